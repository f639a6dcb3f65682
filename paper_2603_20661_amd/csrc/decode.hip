// Decode path (one new token per sequence): embedding, weight-streaming MFMA GEMMs with fused
// RMSNorm scale / rotary + KV-cache write / SwiGLU / residual epilogues, split-KV paged attention,
// argmax.  Activations travel between kernels as hi/lo fp16 pairs already laid out as MFMA B
// operands, so every GEMM's inner loop is loads and MFMAs only.
#include <stdlib.h>

#include <vector>

#include "decode_gemm.h"

// ------------------------------------------------------------------------------------------------
// Plan of the decode attention, built once per step and used by every layer.
//
// The keys of the batch are counted in pairs of 16-key blocks.  All (sequence b, kv head j, pair) triples, in that
// order, form one long list of T = Hkv * sum_b P_b entries (P_b = pairs of sequence b); the attention kernel runs W
// wavefronts and wavefront w takes the entries [w*C, (w+1)*C), C = ceil(T / W), at least min(16, ceil(longest P / 64)).  Every wavefront therefore
// streams the same number of bytes and all of them finish together, whatever the mix of sequence lengths.  A chunk may
// end inside a (b, j) sequence and continue into the next one; each piece is a segment with its own softmax state,
// parked as a record and merged afterwards.  Only the first and the last segment of a chunk can be part of a longer
// sequence, so wavefront w owns the records 2w (the segment its chunk begins with) and 2w + 1 (a later one).
// The cut points depend on the lengths of all sequences of the batch: results are reproducible for a given batch
// but the rounding of a sequence's attention output may differ between batches of different composition.
// C has no other lower bound: with few tokens in the batch a chunk is a single pair, and the whole GPU works on it.  (At
// least 16 pairs a chunk, one sequence of 1041 tokens had 17 wavefronts: 32 us per layer of the 8B shape against 6; a
// step took 4197 us, 3835 with at least 8 pairs, 3661 with 4, 3543 with 1.)  A sequence of up to 32 768 tokens is cut into
// at most 64 full chunks, because the merge reads these in one or two memory round trips (a step of one sequence with 64 chunks
// and with one per wavefront, us: 4096 tokens 3762 / 3877, 8192 3862 / 4014, 16 384 4058 / 4120, 32 768 4467 / 4475).  Beyond, the
// wavefronts that this leaves without work cost more than a round trip (65 536: 5325 / 5122, 131 072: 7027 / 6410), so chunks
// of 16 pairs are long enough.
//   hdr[0] = T, hdr[1] = C;  start[w] = (b, j, first pair, length of b) of wavefront w, b = -1 if it has no work;
//   pref[b] = sum of P over the sequences before b
struct AttnPlan {
  const int32_t* seq_lens;
  int batch, Hkv, W;
  int32_t *hdr, *start, *pref;
};
__device__ __forceinline__ void attn_plan(const AttnPlan& a, int* pref /* LDS: [batch + 1] and the longest P */) {
  const int32_t* __restrict__ const seq_lens = a.seq_lens;
  int32_t *__restrict__ const hdr = a.hdr, *__restrict__ const start = a.start, *__restrict__ const pref_out = a.pref;
  const int batch = a.batch, Hkv = a.Hkv, W = a.W;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < 64) {
    int carry = 0, top = 0;
    if (lane == 0) pref[0] = 0;
    for (int c = 0; c < batch; c += 64) {
      const int bb = c + lane;
      const int P = bb < batch ? max(0, (seq_lens[bb] + 31) / 32) : 0;
      int inc = P;
      top = max(top, P);
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(inc, o);
        if (lane >= o) inc += up;
      }
      if (bb < batch) pref[bb + 1] = carry + inc;
      carry += __shfl(inc, 63);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
    if (lane == 0) pref[batch + 1] = top;
  }
  __syncthreads();
  const int T = pref[batch] * Hkv, longest = pref[batch + 1];
  const int C = max(1, max((T + W - 1) / W, min(16, (longest + 63) / 64)));
  if (tid == 0) { hdr[0] = T; hdr[1] = C; }
  for (int i = tid; i <= batch; i += 256) pref_out[i] = pref[i];
  for (int w = tid; w < W; w += 256) {
    const int64_t x0 = (int64_t)w * C;
    int sb = -1, sj = 0, sp = 0, sctx = 0;
    if (x0 < T) {
      int lo = 0, hi = batch - 1;  // largest b with Hkv * pref[b] <= x0
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)pref[mid] * Hkv <= x0) lo = mid; else hi = mid - 1;
      }
      const int P = max(1, pref[lo + 1] - pref[lo]);  // (never 0 for the sequence that holds entry x0 < T)
      const int r = (int)(x0 - (int64_t)pref[lo] * Hkv);
      sb = lo; sj = r / P; sp = r % P; sctx = seq_lens[lo];
    }
    start[4 * w] = sb; start[4 * w + 1] = sj; start[4 * w + 2] = sp; start[4 * w + 3] = sctx;
  }
}
__global__ __launch_bounds__(256) void attn_plan_kernel(const AttnPlan a) {
  extern __shared__ int plan_lds[];
  attn_plan(a, plan_lds);
}

// ------------------------------------------------------------------------------------------------
// Embedding gather: h = E[token]; sum of squares; packed (h * gain) for the first QKV GEMM.  Workgroup 0 makes the attention's
// plan meanwhile, which needs none of it (a launch of its own: 4.6 us of a step of the tiny shape's 74).
template <typename ET>
__global__ __launch_bounds__(256) void embed_pack_kernel(const int32_t* __restrict__ tokens, const ET* __restrict__ embed, int d,
                                                          const float* __restrict__ gain, float* __restrict__ h,
                                                          float* __restrict__ ssq, uint16_t* __restrict__ xq, int MT, const AttnPlan plan) {
  extern __shared__ int plan_lds[];  // the plan's, or 256 partial sums
  if (blockIdx.x == 0) {
    attn_plan(plan, plan_lds);
    return;
  }
  int t = blockIdx.x - 1;
  const ET* row = embed + (int64_t)tokens[t] * d;
  float local = 0.f;
  for (int o = threadIdx.x; o < d / 8; o += blockDim.x) {
    int k = o * 8;
    union { uint16_t s[8]; u32x4 v; } hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x;
      if constexpr (sizeof(ET) == 4) x = (float)row[k + e];
      else x = bf16_bits_to_float(((const uint16_t*)row)[k + e]);
      h[(int64_t)t * d + k + e] = x;
      local += x * x;
      split_f16(x * gain[k + e], hi.s[e], lo.s[e]);
    }
    *reinterpret_cast<u32x4*>(xq + packed_x_offset(k, t, MT, 0)) = hi.v;
    *reinterpret_cast<u32x4*>(xq + packed_x_offset(k, t, MT, 1)) = lo.v;
  }
  float* red = reinterpret_cast<float*>(plan_lds);
  red[threadIdx.x] = local;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) ssq[(int64_t)t * (MT <= 2 ? SSQ_ROWS : SSQ_TILES)] = red[0];  // row t of the [token][row tile] table; one entry in use
}

// ------------------------------------------------------------------------------------------------
// Skinny GEMM: Y^T[n][t] = sum_k W[n][k] X[t][k] for up to 128 tokens per workgroup pass.
// KH = 1: four wavefronts, each multiplies its two row groups with all four k blocks of a chunk.  KH = 2: eight
// wavefronts (two per SIMD); wavefront w and w + 4 own the same two row groups and take k blocks 0,1 / 2,3 of every
// chunk, so each issues half of the MFMAs and one can issue while its SIMD partner waits for memory; the two partial
// tiles are added through LDS behind the loop and wavefronts 4..7 retire.
template <int MTK, int WMODE, int EPI, int KH>
__global__ __launch_bounds__(256 * KH, MTK == 8 ? 1 : 2 / KH) void skinny_gemm_kernel(const GemmP p) {
  constexpr bool WSPLIT = WMODE == WMODE_SPLIT, W8 = WMODE == WMODE_FP8, W4 = WMODE == WMODE_INT4;
  constexpr int R = 2, KC = 4, WP = WSPLIT ? 2 : 1;
  constexpr int NT = 256 * KH;                     // threads
  constexpr int KPW = KC / KH;                     // k blocks of a chunk per wavefront
  static_assert(KH == 1 || KH == 2);
  constexpr int CHUNK_UNITS = KC * MTK * 128;      // 16-byte units of activations per k chunk
  constexpr int NSTG = (CHUNK_UNITS + NT - 1) / NT;
  __shared__ u32x4 lds[2][CHUNK_UNITS];
  __shared__ float s_scale[MTK * 16];
  // after the main loop the staging buffers are dead and are reused for the epilogue's small reductions
  float(*red)[MTK * 16] = reinterpret_cast<float(*)[MTK * 16]>(&lds[0][0]);
  volatile int* s_last = reinterpret_cast<volatile int*>(&lds[1][0]);

  const int tid = threadIdx.x, wave = (tid >> 6) & 3, khalf = KH == 1 ? 0 : tid >> 8, lane = tid & 63;
  const int k_first = khalf * KPW;                 // first k block of a chunk this wavefront multiplies
  // Workgroup id -> work item.  Consecutive workgroup ids are dealt round-robin to the XCDs (8 here; any power of two
  // up to 8 divides 8), so ids that are equal modulo 8 run behind the same L2.  All k splits of a row tile get such
  // ids: id = c + 8 * slot for row tile c + 8 * lt.  Their partial tiles then meet in one L2 and the split-K hand-over
  // needs no L2 write-back.  Order of the slots: token groups (zb) outermost, then row tiles, then splits; in the two wide
  // GEMMs (gate/up, output head), whose grids are several rounds long, token groups innermost: they run side by side behind
  // one L2 and share the weights (128 tokens in two groups of 64: output head of the 8B shape 407 -> 308 us).
  // The host checks this placement rule with a probe
  // kernel when a model is loaded and sets fence_handover when it does not hold.
  const int slot = blockIdx.x >> 3;
  constexpr bool WIDE = EPI == EPI_SWIGLU || EPI == EPI_LOGITS;
  const int tiles_per_xcd = (p.row_tiles + 7) / 8;
  const int zb = WIDE ? slot % p.zbs : slot / (p.ksplit * tiles_per_xcd);
  const int in_zb = WIDE ? slot / p.zbs : slot % (p.ksplit * tiles_per_xcd);
  const int split = in_zb % p.ksplit, lt = in_zb / p.ksplit;
  const int tile = (blockIdx.x & 7) + 8 * lt;
  if (tile >= p.row_tiles) return;  // grid padding when the row tiles are not a multiple of 8
  const int tb0 = zb * MTK;
  const int rg0 = tile * 8 + wave * R;
  const int kb_begin = split * p.kb_per_split;
  const int kb_end = min(p.KB, kb_begin + p.kb_per_split);
  const int nchunks = (kb_end - kb_begin + KC - 1) / KC;

  int rgc[R];  // clamped row group (loads stay in bounds; stores are masked)
#pragma unroll
  for (int r = 0; r < R; ++r) rgc[r] = min(rg0 + r, p.NRG - 1);

  f32x4 acc[R][MTK];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) acc[r][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Inputs of the epilogue that hang off dependent loads (RMSNorm scale; position and KV block of each token) are
  // requested at kernel entry together with the first weights and activations, and only touched once that first chunk
  // has arrived, so they never put a memory round trip in front of the streaming loop.
  // Sum of squares of a token, the same in every workgroup (a fixed order).  More than 32 tokens (at most 64 entries, one per
  // 128-row tile): wavefront w owns token group w (and w + 4), lane group g = lane/16 reads entries 16g .. 16g+15 of the
  // token's row (four 16-byte loads, always in bounds; entries past n_ssq_in are masked), adds them in index order, and the
  // four groups are combined by two cross-lane exchanges.  Up to 32 tokens (one entry per row group of 16, from
  // small_gemm_kernel): 16 / MTK neighbouring threads read a token's entries, 4 MTK 16-byte pieces each, which covers
  // d_model = 4096, and exchange their sums.
  constexpr bool SQ_ROWS = MTK <= 2;
  constexpr int SUB = 16 / (SQ_ROWS ? MTK : 1), NPC = SQ_ROWS ? 4 * MTK : 1;
  constexpr int NSQ = (MTK + 3) / 4;
  f32x4 ssq_raw[NSQ][4], sq_rows[NPC];
  int pos_pre[MTK];
  int tok_c[MTK];
#pragma unroll
  for (int tb = 0; tb < MTK; ++tb) {
    tok_c[tb] = min((tb0 + tb) * 16 + (lane & 15), p.M - 1);
    pos_pre[tb] = 0;
    if constexpr (EPI == EPI_QKV) pos_pre[tb] = p.seq_lens[tok_c[tb]] - 1;
  }
  const float* sq_row = p.ssq_in + (int64_t)min(tb0 * 16 + tid / SUB, p.M - 1) * SSQ_ROWS;
  if constexpr (SQ_ROWS) {
    if (p.ssq_in && khalf == 0) {
#pragma unroll
      for (int i = 0; i < NPC; ++i) sq_rows[i] = *reinterpret_cast<const f32x4*>(sq_row + (i * SUB + tid % SUB) * 4);
    }
  } else if (p.ssq_in && wave < MTK && khalf == 0) {
#pragma unroll
    for (int q = 0; q < NSQ; ++q) {
      const int t = min((tb0 + wave + 4 * q) * 16 + (lane & 15), p.M - 1);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        ssq_raw[q][c] = *reinterpret_cast<const f32x4*>(p.ssq_in + (int64_t)t * SSQ_TILES + (lane >> 4) * 16 + c * 4);
    }
  }
  float scale_pre[MTK];
  int blk_pre[MTK];
  // before the first barrier: reduce the sums and publish the scales; table loads for the KV slots go out
  auto finish_prefetch = [&]() __attribute__((always_inline)) {
    if constexpr (SQ_ROWS) {
      if (p.ssq_in && khalf == 0) {
        float s = 0.f;
        auto add = [&](f32x4 v, int e0) __attribute__((always_inline)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) s += e0 + e < p.n_ssq_in ? v[e] : 0.f;
        };
#pragma unroll
        for (int i = 0; i < NPC; ++i) add(sq_rows[i], (i * SUB + tid % SUB) * 4);
        for (int i = NPC; i * SUB * 4 < p.n_ssq_in; ++i)
          add(*reinterpret_cast<const f32x4*>(sq_row + (i * SUB + tid % SUB) * 4), (i * SUB + tid % SUB) * 4);
#pragma unroll
        for (int o = SUB / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (tid % SUB == 0) s_scale[tid / SUB] = rsqrtf(s * p.inv_dim + p.eps);
      }
    } else if (p.ssq_in && wave < MTK && khalf == 0) {
#pragma unroll
      for (int q = 0; q < NSQ; ++q) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) s += ((lane >> 4) * 16 + c * 4 + e < p.n_ssq_in) ? ssq_raw[q][c][e] : 0.f;
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < 16) s_scale[(wave + 4 * q) * 16 + lane] = rsqrtf(s * p.inv_dim + p.eps);
      }
    }
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      blk_pre[tb] = 0;
      if constexpr (EPI == EPI_QKV) blk_pre[tb] = kv_block_id(p.table + (int64_t)tok_c[tb] * p.mbs, pos_pre[tb]);
    }
  };
  // after that barrier
  auto read_scales = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      scale_pre[tb] = p.ssq_in ? s_scale[tb * 16 + (lane & 15)] : 1.f;
      if constexpr (W8) scale_pre[tb] *= p.wfactor;
    }
  };

  u32x4 wA[KC][R][WP], wB[KC][R][WP], stg[NSTG];
  const int last_tb = (p.M - 1) / 16 - tb0;  // last token group of this workgroup that holds a sequence

  // Loads past the end of this split's k range are redirected to its last valid block (in bounds) and the
  // matching MFMAs are skipped in compute(): no per-element selects in the streaming loop.
  auto load_w = [&](u32x4(&w)[KC][R][WP], int c) {
    if constexpr (W4) {
      // one 16-byte unit carries the whole chunk (entry 0 of the set); entry 1 takes the four group scales (8 bytes)
      const int chunk = min((kb_begin + c * KC) >> 2, (kb_end - 1) >> 2);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t unit = ((int64_t)chunk * p.NRG + rgc[r]) * 64 + lane, scale = ((int64_t)chunk * p.NRG + rgc[r]) * 16 + (lane & 15);
        if constexpr (KH == 1) {
          w[0][r][0] = p.W[unit];
          const u32x2 sc = p.Wscale[scale];
          w[1][r][0] = u32x4{sc.x, sc.y, 0u, 0u};
        } else {  // only the half of the unit (two k blocks) and the two scales this wavefront multiplies
          const u32x2 half = reinterpret_cast<const u32x2*>(p.W)[unit * 2 + khalf];
          w[0][r][0] = u32x4{half.x, half.y, 0u, 0u};
          w[1][r][0] = u32x4{reinterpret_cast<const uint32_t*>(p.Wscale)[scale * 2 + khalf], 0u, 0u, 0u};
        }
      }
      return;
    }
    if constexpr (W8) {
      // one 16-byte unit carries two k blocks: entries 0 and 2 of the set hold the chunk's two units, 1 and 3 stay unused
      // (kb_begin is a multiple of 4, so a chunk starts on a pair)
#pragma unroll
      for (int j = 0; j < KPW; j += 2) {
        const int pair = min((kb_begin + c * KC + k_first + j) >> 1, (kb_end - 1) >> 1);
#pragma unroll
        for (int r = 0; r < R; ++r) w[j][r][0] = p.W[((int64_t)pair * p.NRG + rgc[r]) * 64 + lane];
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < KPW; ++j) {  // register slot j holds k block k_first + j of the chunk
      const int kbc = min(kb_begin + c * KC + k_first + j, kb_end - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t idx = ((int64_t)kbc * p.NRG + rgc[r]) * 64 + lane;
        w[j][r][0] = p.W[idx];
        if constexpr (WSPLIT) w[j][r][1] = p.Wlo[idx];
      }
    }
  };
  auto load_stage = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) {
      const int u = min(tid + i * NT, CHUNK_UNITS - 1);  // (more threads than units when MTK = 1 and KH = 2)
      // (token groups past the last sequence: its group again, in L1 by then; their columns of the result are dropped)
      const int kk = u / (MTK * 128), within = min(u % (MTK * 128) / 128, last_tb) * 128 + u % 128;
      const int kbc = min(kb_begin + c * KC + kk, kb_end - 1);
      stg[i] = p.X[((int64_t)kbc * p.MT + tb0) * 128 + within];
    }
  };
  auto store_stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) lds[buf][min(tid + i * NT, CHUNK_UNITS - 1)] = stg[i];
  };
  // nvalid = k blocks of the chunk that lie inside the range: KC for every chunk but possibly the last.
  // The B fragments (activations) of the next up to four token groups are fetched from LDS while the MFMAs of the current
  // ones run.
  auto compute = [&](u32x4(&w)[KC][R][WP], int buf, int nvalid) __attribute__((always_inline)) {
    constexpr int TG = MTK < 4 ? MTK : 4, NG = MTK / TG;
    u32x4 bq[2][TG][2];
    auto fetch = [&](int set, int kk, int grp) __attribute__((always_inline)) {
#pragma unroll
      for (int tb = 0; tb < TG; ++tb) {
        bq[set][tb][0] = lds[buf][(kk * MTK + grp * TG + tb) * 128 + lane];
        bq[set][tb][1] = lds[buf][(kk * MTK + grp * TG + tb) * 128 + 64 + lane];
      }
    };
    fetch(0, k_first, 0);
    f16x8 a8[R];
#pragma unroll
    for (int st = 0; st < KPW * NG; ++st) {
      const int j = st / NG, grp = st % NG;  // k block k_first + j of the chunk, operands in register slot j; token groups TG grp ..
      if (k_first + j >= nvalid) break;
      if (st + 1 < KPW * NG) fetch((st + 1) & 1, k_first + (st + 1) / NG, (st + 1) % NG);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (W8) {
        if (grp == 0) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const u32x4 raw = w[j & ~1][r][0];
            a8[r] = (j & 1) ? fp8x8_to_f16x8(raw.z, raw.w) : fp8x8_to_f16x8(raw.x, raw.y);
          }
        }
      }
      if constexpr (W4) {  // (j is the k block of the unit, or of its half)
        if (grp == 0) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const u32x4 raw = w[0][r][0], sc = w[1][r][0];
            const uint32_t word = j == 0 ? raw.x : j == 1 ? raw.y : j == 2 ? raw.z : raw.w;
            const uint32_t s2 = j < 2 ? sc.x : sc.y;
            const uint32_t s16 = (j & 1) ? (s2 >> 16) : (s2 & 0xFFFFu);
            a8[r] = int4x8_to_f16x8(word, __builtin_bit_cast(f16x2, s16 | (s16 << 16)));
          }
        }
      }
#pragma unroll
      for (int tb = 0; tb < TG; ++tb) {
        const f16x8 bhi = as_f16x8(bq[st & 1][tb][0]), blo = as_f16x8(bq[st & 1][tb][1]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          f32x4& c = acc[r][grp * TG + tb];
          f16x8 a;
          if constexpr (W8 || W4) a = a8[r];
          else a = as_f16x8(w[j][r][0]);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bhi, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, blo, c, 0, 0, 0);
          if constexpr (WSPLIT) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(w[j][r][1]), bhi, c, 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Software pipeline: while chunk c is multiplied out of LDS buffer c&1 and register set A/B, chunk c+1 is
  // already on its way from HBM.  The steady-state loop has no conditional loads, so the new loads can stay
  // in flight across the MFMAs of the current chunk; the last one or two chunks are peeled.
  if (nchunks > 0) {
    const int last_valid = (kb_end - kb_begin) - (nchunks - 1) * KC;  // k blocks in the final chunk
    load_stage(0);
    load_w(wA, 0);
    __builtin_amdgcn_sched_barrier(0);
    store_stage(0);
    finish_prefetch();
    __syncthreads();
    read_scales();
    int c = 0;
    for (; c + 2 < nchunks; c += 2) {
      load_stage(c + 1);
      load_w(wB, c + 1);
      __builtin_amdgcn_sched_barrier(0);  // keep the prefetch in front of the MFMAs it overlaps with
      compute(wA, 0, KC);
      __builtin_amdgcn_sched_barrier(0);
      store_stage(1);
      __syncthreads();
      load_stage(c + 2);
      load_w(wA, c + 2);
      __builtin_amdgcn_sched_barrier(0);
      compute(wB, 1, KC);
      __builtin_amdgcn_sched_barrier(0);
      store_stage(0);
      __syncthreads();
    }
    if (c + 1 < nchunks) {
      load_stage(c + 1);
      load_w(wB, c + 1);
      __builtin_amdgcn_sched_barrier(0);
      compute(wA, 0, KC);
      __builtin_amdgcn_sched_barrier(0);
      store_stage(1);
      __syncthreads();
      compute(wB, 1, last_valid);
    } else {
      compute(wA, 0, last_valid);
    }
    __syncthreads();
  } else {
    finish_prefetch();
    __syncthreads();
    read_scales();
  }

  if constexpr (KH == 2) {
    // the staging buffers are dead: wavefronts 4..7 hand their partial tile to wavefronts 0..3 (same rows) and retire;
    // the barriers further down then only count the wavefronts that are left
    u32x4* xch = &lds[0][0];  // [wavefront 0..3][r][tb][lane]
    if (khalf == 1) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int tb = 0; tb < MTK; ++tb) xch[((wave * R + r) * MTK + tb) * 64 + lane] = __builtin_bit_cast(u32x4, acc[r][tb]);
    }
    __syncthreads();
    if (khalf == 1) return;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) acc[r][tb] += __builtin_bit_cast(f32x4, xch[((wave * R + r) * MTK + tb) * 64 + lane]);
    __syncthreads();  // `red` and `s_last` below reuse the same LDS
  }

  // accumulator layout: acc[r][tb][i] = Y^T[row][token], row = (rg0+r)*16 + (lane/16)*4 + i, token = (tb0+tb)*16 + lane%16
  const int rsub = (lane >> 4) * 4;
  const int tsub = lane & 15;

  // Operands of the epilogue that live in memory (residual stream and next norm's gain; rotary factors) are requested
  // before the split-K partial tiles, so the last workgroup pays one memory round trip for everything it needs.
  // Addresses are clamped into range; values of invalid rows / tokens are never used.
  f32x4 hv_pre[R][MTK], gv_pre[R], cs_pre[R][MTK];
  auto request_epilogue_inputs = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int n0 = rgc[r] * 16 + rsub;
      if constexpr (EPI == EPI_RESID) gv_pre[r] = *reinterpret_cast<const f32x4*>(p.gain_next + n0);
      if constexpr (EPI == EPI_QKV) {  // gains of the head normalisation (value rows read the key gains and ignore them)
        if (p.qk_gain) gv_pre[r] = *reinterpret_cast<const f32x4*>(p.qk_gain + (n0 / p.hd < p.Hq ? 0 : p.hd) + n0 % p.hd);
      }
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) {
        if constexpr (EPI == EPI_RESID) hv_pre[r][tb] = *reinterpret_cast<const f32x4*>(p.h + (int64_t)tok_c[tb] * p.d + n0);
        if constexpr (EPI == EPI_QKV)
          cs_pre[r][tb] = *reinterpret_cast<const f32x4*>(p.rope + (int64_t)pos_pre[tb] * (p.hd / 2) + ((n0 % p.hd) >> 1));
      }
    }
  };

  if (p.ksplit <= 1) request_epilogue_inputs();
  if (MTK < 8 && p.ksplit > 1) {
    // split-K: park the partial tile, and let the workgroup that arrives last add all partial tiles in split order
    // parked as a register image: unit ((((split, zb, tile), wave), r), tb), lane -> one 16-byte store per lane,
    // 1 KiB contiguous per instruction; the last workgroup reads it back with the same thread mapping
    const __amdgpu_buffer_rsrc_t prs = shared_rsrc(p.partial);
    auto punit = [&](int sp, int r, int tb) __attribute__((always_inline)) {
      return (uint32_t)((((((sp * p.zbs + zb) * p.row_tiles + tile) * 4 + wave) * R + r) * MTK + tb) * 64 + lane) * 16u;
    };
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) store_shared_f32x4(prs, punit(split, r, tb), acc[r][tb]);
    wait_own_memory_ops();
    __syncthreads();
    if (tid == 0) *s_last = arrive_last(&p.counters[zb * p.row_tiles + tile], p.ksplit, p.fence_handover, p.fault_flag);
    __syncthreads();
    if (!*s_last) return;
    // the fenced hand-over's other half: the partial tiles may come from another L2, so everything this workgroup has
    // cached is dropped before they are read (acquire side of the producers' release fences)
    if (p.fence_handover) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid == 0) __hip_atomic_store(&p.counters[zb * p.row_tiles + tile], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    request_epilogue_inputs();
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) acc[r][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Partial tiles are added in split order (reproducible), four on their way at a time.  In batches in the fp32 residual and
    // gate/up kernels of 64 tokens, whose registers are full: with the ring they spill 92 and 83 registers instead of 78 and 74, in
    // the main loop too (8B shape, 48 sequences: O 39.7 -> 36.6 us, gate/up 164 -> 147, down 89 -> 84, a step of 6 layers 2852 ->
    // 2694; the QKV and head kernels spill less with the ring, 118 and 70 against 126 and 74).
    constexpr int NSP = 4;
    if constexpr (WSPLIT && MTK == 4 && (EPI == EPI_RESID || EPI == EPI_SWIGLU)) {
      for (int s0 = 0; s0 < p.ksplit; s0 += NSP) {
        f32x4 pv[NSP][R][MTK];
#pragma unroll
        for (int u = 0; u < NSP; ++u) {
          const int sidx = min(s0 + u, p.ksplit - 1);
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int tb = 0; tb < MTK; ++tb) pv[u][r][tb] = load_shared_f32x4(prs, punit(sidx, r, tb));
        }
#pragma unroll
        for (int u = 0; u < NSP; ++u) {
          if (s0 + u >= p.ksplit) break;
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int tb = 0; tb < MTK; ++tb) acc[r][tb] += pv[u][r][tb];
        }
      }
    } else {
      f32x4 pv[NSP][R][MTK];
      add_in_order<NSP>(p.ksplit,
          [&](int u, int sp) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
              for (int tb = 0; tb < MTK; ++tb) pv[u][r][tb] = load_shared_f32x4(prs, punit(sp, r, tb));
          },
          [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
              for (int tb = 0; tb < MTK; ++tb) acc[r][tb] += pv[u][r][tb];
          });
    }
  }

  float ssq_local[MTK];
#pragma unroll
  for (int tb = 0; tb < MTK; ++tb) ssq_local[tb] = 0.f;
  float best[EPI == EPI_LOGITS ? MTK : 1];
  int best_at[EPI == EPI_LOGITS ? MTK : 1];

  // Normalised query / key heads: 1 / rms of each token's head vector.  A row tile holds whole heads (128 rows: one head
  // of 128, or two of 64 owned by wavefronts 0,1 and 2,3); a wavefront adds the squares of its 32 rows per token (lanes,
  // then two cross-lane exchanges) and the wavefronts of a head are added through LDS in index order.  Row groups past
  // the end of the matrix only ever fall into a head that does not exist.
  float head_rs[MTK];
  if constexpr (EPI == EPI_QKV) {
    if (p.qk_gain) {
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) {
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = acc[r][tb][i] * scale_pre[tb];
            s += v * v;
          }
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < 16) red[wave][tb * 16 + lane] = s;
      }
      __syncthreads();
#pragma unroll
      for (int tb = 0; tb < MTK; ++tb) {
        const int at = tb * 16 + tsub;
        const float tot = p.hd == 128 ? (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]) : red[wave & 2][at] + red[(wave & 2) + 1][at];
        head_rs[tb] = rsqrtf(tot / (float)p.hd + p.eps);
      }
    }
  }

  // QKV: finish the values in place (RMSNorm factor, head normalisation, rotation), then take, per token, the largest
  // magnitude of every head's vector (lanes, two cross-lane exchanges, the head's wavefronts through LDS): the scale of
  // the key / value codes.  (Query heads get one too and ignore it.)
  float head_amax[MTK];
  if constexpr (EPI == EPI_QKV) {
    const int rot_rows = (p.Hq + p.Hkv) * p.hd;
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      float am = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int n0 = (rg0 + r) * 16 + rsub;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[r][tb][i] * scale_pre[tb];
        if (n0 < rot_rows) {
          if (p.qk_gain) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= head_rs[tb] * gv_pre[r][i];
          }
          // rows arrive with the rotary pair (i, i + hd/2) at neighbouring positions (2i, 2i+1)
#pragma unroll
          for (int pr = 0; pr < 2; ++pr) {
            const float cs_x = cs_pre[r][tb][2 * pr], cs_y = cs_pre[r][tb][2 * pr + 1];
            float a = v[2 * pr], b = v[2 * pr + 1];
            v[2 * pr] = a * cs_x - b * cs_y;
            v[2 * pr + 1] = b * cs_x + a * cs_y;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[r][tb][i] = v[i];
          am = fmaxf(am, __builtin_fabsf(v[i]));  // (a NaN element is dropped by fmaxf; its code is 0)
        }
      }
      am = fmaxf(am, __shfl_xor(am, 16));
      am = fmaxf(am, __shfl_xor(am, 32));
      head_amax[tb] = am;
    }
    if (p.qk_gain) __syncthreads();  // `red` may still be read by the head normalisation above
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb)
      if (lane < 16) red[wave][tb * 16 + lane] = head_amax[tb];
    __syncthreads();
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      const int at = tb * 16 + tsub;
      head_amax[tb] = p.hd == 128 ? fmaxf(fmaxf(red[0][at], red[1][at]), fmaxf(red[2][at], red[3][at]))
                                  : fmaxf(red[wave & 2][at], red[(wave & 2) + 1][at]);
    }
  }

#pragma unroll
  for (int tb = 0; tb < MTK; ++tb) {
    const int t = (tb0 + tb) * 16 + tsub;
    const bool tok_ok = t < p.M;
    const float scale = scale_pre[tb];

    if constexpr (EPI == EPI_LOGITS) { best[tb] = NEG_INF; best_at[tb] = 0x7fffffff; }
    if constexpr (EPI == EPI_SWIGLU) {
      if (tok_ok && rg0 + 1 < p.NRG) {
        int f0 = (rg0 >> 1) * 16 + rsub;
        union { uint16_t s[4]; u32x2 v; } hi, lo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float g = acc[0][tb][i] * scale, u = acc[1][tb][i] * scale;
          float a = g / (1.f + __expf(-g)) * u;
          split_f16(a, hi.s[i], lo.s[i]);
        }
        *reinterpret_cast<u32x2*>(p.xa + packed_x_offset(f0, t, p.MT, 0)) = hi.v;
        *reinterpret_cast<u32x2*>(p.xa + packed_x_offset(f0, t, p.MT, 1)) = lo.v;
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!tok_ok || rg0 + r >= p.NRG) continue;
        const int n0 = (rg0 + r) * 16 + rsub;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[r][tb][i] * scale;  // (QKV: overwritten below, the values are already final)

        if constexpr (EPI == EPI_LOGITS) {
          *reinterpret_cast<float4*>(p.logits + (int64_t)t * p.V + n0) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
          for (int i = 0; i < 4; ++i) argmax_take(best[tb], best_at[tb], v[i], n0 + i);
        } else if constexpr (EPI == EPI_RESID) {
          const f32x4 hv = hv_pre[r][tb], gv = gv_pre[r];
          float hn[4] = {hv[0] + v[0], hv[1] + v[1], hv[2] + v[2], hv[3] + v[3]};
          float gn[4] = {gv[0], gv[1], gv[2], gv[3]};
          *reinterpret_cast<float4*>(p.h + (int64_t)t * p.d + n0) = make_float4(hn[0], hn[1], hn[2], hn[3]);
          union { uint16_t s[4]; u32x2 v; } hi, lo;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ssq_local[tb] += hn[i] * hn[i];
            split_f16(hn[i] * gn[i], hi.s[i], lo.s[i]);
          }
          *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, p.MT, 0)) = hi.v;
          *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, p.MT, 1)) = lo.v;
        } else {  // EPI_QKV: the values were finished (scaled, normalised, rotated) in place above
          const int head = n0 / p.hd, c0 = n0 % p.hd;
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = acc[r][tb][i];
          if (head < p.Hq) {
            // queries leave as fp16 hi + lo, already multiplied by log2(e)/sqrt(hd), in the order the attention kernel loads them
            union { uint16_t s[4]; u32x2 v; } qh, ql;
#pragma unroll
            for (int i = 0; i < 4; ++i) split_f16(v[i] * p.qscale, qh.s[i], ql.s[i]);
            *reinterpret_cast<u32x2*>(p.q_hi + (int64_t)t * (p.Hq * p.hd) + n0) = qh.v;
            *reinterpret_cast<u32x2*>(p.q_lo + (int64_t)t * (p.Hq * p.hd) + n0) = ql.v;
          } else {
            // keys and values go to the cache as 16-bit codes with the scale of their (token, head) vector
            const int64_t slot = kv_slot_in_block(blk_pre[tb], pos_pre[tb]);
            const int64_t blk = slot / KV_BS;
            const int tok = (int)(slot % KV_BS);
            const bool is_v = head >= p.Hq + p.Hkv;
            const int j = head - p.Hq - (is_v ? p.Hkv : 0);
            const float inv = kv_code_inv(head_amax[tb]);
            union { uint16_t s[4]; u32x2 v; } code;
#pragma unroll
            for (int i = 0; i < 4; ++i) code.s[i] = kv_code(v[i], inv);
            if (!is_v) {
              *reinterpret_cast<u32x2*>(p.kplane + (blk * p.Hkv + j) * (int64_t)(KV_BS * p.hd) + k_cache_offset(tok, c0)) = code.v;
            } else {
              uint16_t* dst = p.vplane + (blk * p.Hkv + j) * (int64_t)(KV_BS * p.hd);
#pragma unroll
              for (int i = 0; i < 4; ++i) dst[v_cache_offset(tok, c0 + i)] = code.s[i];
            }
            if (c0 == 0 && rsub == 0)  // one lane per (token, head): first row of the head
              p.kvscale[kv_scale_offset(blk, p.Hkv, j) + (is_v ? 16 : 0) + tok] = kv_code_scale(head_amax[tb]);
          }
        }
      }
    }
  }

  if constexpr (EPI == EPI_LOGITS) {  // the largest of this row tile per token, for argmax_kernel
    if (!p.best_val) return;
    int(*at)[MTK * 16] = reinterpret_cast<int(*)[MTK * 16]>(red + 4);
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      argmax_of_rows(best[tb], best_at[tb]);
      if (lane < 16) { red[wave][tb * 16 + lane] = best[tb]; at[wave][tb * 16 + lane] = best_at[tb]; }
    }
    __syncthreads();
    const int t = tb0 * 16 + tid;
    if (tid < MTK * 16 && t < p.M) {
      float b = red[0][tid];
      int i = at[0][tid];
#pragma unroll
      for (int w = 1; w < 4; ++w) argmax_take(b, i, red[w][tid], at[w][tid]);
      p.best_val[(int64_t)t * p.row_tiles + tile] = b;
      p.best_idx[(int64_t)t * p.row_tiles + tile] = i;
    }
  }
  if constexpr (EPI == EPI_RESID) {
    // per (row tile, token) sum of squares of the new residual, reduced in a fixed order
#pragma unroll
    for (int tb = 0; tb < MTK; ++tb) {
      float s = ssq_local[tb];
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < 16) red[wave][tb * 16 + lane] = s;
    }
    __syncthreads();
    if (tid < MTK * 16) {
      int t = tb0 * 16 + tid;
      if (t < p.M) p.ssq_out[(int64_t)t * (SQ_ROWS ? SSQ_ROWS : SSQ_TILES) + tile] = red[0][tid] + red[1][tid] + red[2][tid] + red[3][tid];
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Two 16-bit codes (one 32-bit word, offset binary u = x + 32768) as two pairs of fp16 numbers a, b with x = 256 a + b,
// a in [-128, 127], b in [0, 255] - both exact in fp16, so the matrix cores multiply the codes without losing a bit.
// The high and low bytes of u are planted in the mantissa of the fp16 number 1024 (0x6400 | n = 1024 + n) and
// 1024 + 128, resp. 1024, is subtracted, two values per instruction.
__device__ __forceinline__ void split_codes(uint32_t u, uint32_t& hi, uint32_t& lo) {
  const f16x2 off_hi = {(_Float16)1152.f, (_Float16)1152.f}, off_lo = {(_Float16)1024.f, (_Float16)1024.f};
  const uint32_t ph = __builtin_amdgcn_perm(0x64646464u, u, 0x04030401u);  // bytes: u.b1, 0x64, u.b3, 0x64
  const uint32_t pl = __builtin_amdgcn_perm(0x64646464u, u, 0x04020400u);  // bytes: u.b0, 0x64, u.b2, 0x64
  hi = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, ph) - off_hi);
  lo = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, pl) - off_lo);
}
__device__ __forceinline__ void split_codes4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, f16x8& hi, f16x8& lo) {
  uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
  split_codes(w0, h0, l0);
  split_codes(w1, h1, l1);
  split_codes(w2, h2, l2);
  split_codes(w3, h3, l3);
  hi = as_f16x8(u32x4{h0, h1, h2, h3});
  lo = as_f16x8(u32x4{l0, l1, l2, l3});
}
__device__ __forceinline__ void split_codes8(u32x4 w, f16x8& hi, f16x8& lo) { split_codes4(w.x, w.y, w.z, w.w, hi, lo); }

// Where column k of sequence b's attention output goes: the decode path's packed operand of the O projection, or (first_row >= 0)
// the rows of a prefill call that its last position rides in (K16 = columns / 16)
__device__ __forceinline__ int64_t attn_out_offset(int k, int b, int hl, int MT, int first_row, int K16) {
  return first_row < 0 ? packed_x_offset(k, b, MT, hl) : packed_p_offset(first_row + (b >> 4) * 32 + hl * 16 + (b & 15), k, K16);
}

// ------------------------------------------------------------------------------------------------
// Decode attention.  Each wavefront walks its chunk of the plan above, segment by segment:
//   S^T = K Q^T (keys x heads), online softmax per head along the key axis with cross-lane shuffles,
//   O^T = V^T P^T (head_dim x heads).  The G query heads of the group share every K/V byte.
// A segment that covers its whole (sequence, kv head) writes the packed hi/lo operand of the O projection itself;
// otherwise it parks (m, l, unnormalised o) in one of its two records.
template <int HD, int G>
__global__ __launch_bounds__(256) void decode_attn_kernel(const uint16_t* __restrict__ q_hi, const uint16_t* __restrict__ q_lo,
                                                           const uint16_t* __restrict__ kplane,
                                                           const uint16_t* __restrict__ vplane, const float* __restrict__ kvscale,
                                                           const int32_t* __restrict__ seq_lens,
                                                           const int32_t* __restrict__ table, int batch, int mbs, int Hq, int Hkv,
                                                           const int32_t* __restrict__ hdr, const int32_t* __restrict__ start,
                                                           float* __restrict__ part, uint16_t* __restrict__ xo, int MT, int first_row) {
  constexpr int NKF = HD / 32;  // K fragments per block
  constexpr int NVF = HD / 16;  // V fragments per block
  constexpr int PSTRIDE = HD + 4;  // floats per (record, head): o[HD], m, l, pad
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = lane & 15, g = lane >> 4;
  // A list shorter than the number of wavefronts is dealt out over the workgroups, so that it still reaches every compute
  // unit; a longer one is not, neighbouring chunks then share a compute unit (64 sequences of the 8B shape: 6385 against
  // 6452 us a step).  Both candidates are requested at once, before the length of the list is known.
  const int w_near = blockIdx.x * 4 + wave, w_far = wave * gridDim.x + blockIdx.x;
  const u32x4 st_near = *reinterpret_cast<const u32x4*>(start + 4 * w_near), st_far = *reinterpret_cast<const u32x4*>(start + 4 * w_far);
  const int T = hdr[0], C = hdr[1];
  const bool far = T < (int)gridDim.x * 4;
  const int w = far ? w_far : w_near;
  const u32x4 st = far ? st_far : st_near;
  int b = __builtin_amdgcn_readfirstlane((int)st.x);
  if (b < 0) return;
  int j = __builtin_amdgcn_readfirstlane((int)st.y);
  int p = __builtin_amdgcn_readfirstlane((int)st.z);
  int ctx = __builtin_amdgcn_readfirstlane((int)st.w);
  int x = w * C;                      // position in the list of the next entry
  int remaining = min(C, T - x);
  const int64_t blk_elems = (int64_t)KV_BS * HD;

  while (remaining > 0 && b < batch) {  // (the second test only guards against a plan that does not match the lengths)
    const int P = (ctx + 31) / 32;
    if (P <= 0) {  // an empty sequence has no entries in the list
      if (++b < batch) ctx = __builtin_amdgcn_readfirstlane(seq_lens[b]);
      continue;
    }
    const int np = min(P - p, remaining);
    const int kend = min(ctx, (p + np) * 32);
    const int32_t* trow = table + (int64_t)b * mbs;
    // Q^T operand: lane (head n, group g) holds dims f*32 + g*8 .. +7 of head n, as fp16 hi + lo (pre-scaled by the producer)
    f16x8 qhi[NKF], qlo[NKF];
    {
      const int64_t qoff = ((int64_t)b * Hq + j * G + min(n, G - 1)) * HD + g * 8;
#pragma unroll
      for (int f = 0; f < NKF; ++f) {
        u32x4 h = *reinterpret_cast<const u32x4*>(q_hi + qoff + f * 32);
        u32x4 l = *reinterpret_cast<const u32x4*>(q_lo + qoff + f * 32);
        if (n >= G) { h = u32x4{0, 0, 0, 0}; l = u32x4{0, 0, 0, 0}; }
        qhi[f] = as_f16x8(h);
        qlo[f] = as_f16x8(l);
      }
    }
    f32x4 oacc[NVF];
#pragma unroll
    for (int f = 0; f < NVF; ++f) oacc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = NEG_INF, l_run = 0.f;
    // The value scales ride on the probabilities (fp16 operands of the second product).  To keep those operands in
    // fp16's normal range whatever the magnitude of the model's values, they are multiplied by a power of two taken
    // from the first key's scale (2^-4 / 2^exponent, so p * scale * vnorm is about p / 16) and the accumulator is
    // divided by it at the end of the segment.  Scales more than 2^11 times the first one would saturate.
    float vnorm = 0.f, vnorm_inv = 0.f;

    // the segment in runs of at most 32 pairs = 64 blocks, whose ids are held one per lane
    for (int sp = 0; sp < np; sp += 32) {
      const int npairs = min(32, np - sp);
      const int k0 = (p + sp) * 32;
      const int blk0 = k0 / KV_BS;
      const int my_blk = trow[min(blk0 + lane, mbs - 1)];
      const int last_blk_local = min(63, (kend - 1) / KV_BS - blk0);  // index, within this run, of its last valid block

      struct KV {
        u32x4 k0[NKF], k1[NKF];
        u32x2 v0[NVF], v1[NVF];
        f32x4 ks0, ks1, vs0, vs1;  // scales of this lane's keys 4g .. 4g+3 of the two blocks
      };
      auto load_pair = [&](KV& r, int pr) __attribute__((always_inline)) {
        const int id0 = __shfl(my_blk, min(2 * pr, last_blk_local));
        const int id1 = __shfl(my_blk, min(2 * pr + 1, last_blk_local));  // past the end: the last block again (masked)
        const int64_t off0 = ((int64_t)id0 * Hkv + j) * blk_elems;
        const int64_t off1 = ((int64_t)id1 * Hkv + j) * blk_elems;
        const float* sc0 = kvscale + kv_scale_offset(id0, Hkv, j) + 4 * g;
        const float* sc1 = kvscale + kv_scale_offset(id1, Hkv, j) + 4 * g;
        r.ks0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(sc0));
        r.vs0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(sc0 + 16));
        r.ks1 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(sc1));
        r.vs1 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(sc1 + 16));
#pragma unroll
        for (int f = 0; f < NKF; ++f) {
          r.k0[f] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kplane + off0 + (f * 64 + lane) * 8));
          r.k1[f] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kplane + off1 + (f * 64 + lane) * 8));
        }
#pragma unroll
        for (int f = 0; f < NVF; ++f) {
          r.v0[f] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(vplane + off0 + (f * 64 + lane) * 4));
          r.v1[f] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(vplane + off1 + (f * 64 + lane) * 4));
        }
      };
      auto process = [&](KV& r, int pr) __attribute__((always_inline)) {
        const int base = k0 + pr * 32;
        // scores (already in log2 units): lane (head n, g) gets keys base + 4g + i (block 0) and base + 16 + 4g + i (block 1).
        // Codes x = 256 a + b: the a plane meets both query planes, the b plane the hi plane (b q_lo is below 2^-19 of the score).
        f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f}, b0 = {0.f, 0.f, 0.f, 0.f}, b1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < NKF; ++f) {
          f16x8 ka, kb;
          split_codes8(r.k0[f], ka, kb);
          a0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qhi[f], a0, 0, 0, 0);
          a0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qlo[f], a0, 0, 0, 0);
          b0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kb, qhi[f], b0, 0, 0, 0);
          split_codes8(r.k1[f], ka, kb);
          a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qhi[f], a1, 0, 0, 0);
          a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qlo[f], a1, 0, 0, 0);
          b1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kb, qhi[f], b1, 0, 0, 0);
        }
        if (vnorm == 0.f) {  // first pair of the segment: its first key is valid, its scale sets the normaliser
          const uint32_t bits = __builtin_amdgcn_readfirstlane(__float_as_uint(r.vs0[0]));
          int e = (int)((bits >> 23) & 0xffu);
          e = e < 8 ? 114 : min(e, 240);  // an all-zero first value vector: take 2^-13; (NaN / inf: anything finite)
          vnorm = __uint_as_float((uint32_t)(250 - e) << 23);           // 2^(123 - e): scale * vnorm lies in [1/16, 1/8)
          vnorm_inv = __uint_as_float((uint32_t)(e + 4) << 23);         // 2^(e - 123)
        }
        float sc[8], pvs[8];
        float mx = NEG_INF;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool ok0 = base + 4 * g + i < kend, ok1 = base + 16 + 4 * g + i < kend;
          sc[i] = ok0 ? (a0[i] * 256.f + b0[i]) * r.ks0[i] : NEG_INF;
          sc[4 + i] = ok1 ? (a1[i] * 256.f + b1[i]) * r.ks1[i] : NEG_INF;
          pvs[i] = ok0 ? r.vs0[i] * vnorm : 0.f;      // slots past the end may hold anything: their scale never enters
          pvs[4 + i] = ok1 ? r.vs1[i] * vnorm : 0.f;
          mx = fmaxf(mx, fmaxf(sc[i], sc[4 + i]));
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float ref = m_new == NEG_INF ? 0.f : m_new;  // (scores of -inf only, so far: no weight, and not a NaN)
        const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
        // the probabilities times the value scales go to the matrix cores as fp16 hi + lo, like every other operand of the
        // single-token path (for the a plane of the value codes with the factor 256; the b plane, 2^-8 of the value, takes
        // the hi part alone); non-negative, so one bound keeps a wild scale from overflowing
        union { _Float16 s[8]; f16x8 v; } pa, pl, pb;
        float psum = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float pv = __builtin_amdgcn_exp2f(sc[i] - ref);
          psum += pv;
          const float w = fminf(pv * pvs[i], 255.f), w256 = w * 256.f;
          pa.s[i] = (_Float16)w256;
          pl.s[i] = (_Float16)(w256 - (float)pa.s[i]);
          pb.s[i] = (_Float16)w;
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
        if (__any(alpha != 1.f)) {  // the running maximum moved for some head of the wavefront (rare after the first pairs)
#pragma unroll
          for (int f = 0; f < NVF; ++f) {
            oacc[f][0] *= alpha; oacc[f][1] *= alpha; oacc[f][2] *= alpha; oacc[f][3] *= alpha;
          }
        }
#pragma unroll
        for (int f = 0; f < NVF; ++f) {
          f16x8 va, vb;
          split_codes4(r.v0[f].x, r.v0[f].y, r.v1[f].x, r.v1[f].y, va, vb);
          oacc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, pa.v, oacc[f], 0, 0, 0);
          oacc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, pl.v, oacc[f], 0, 0, 0);
          oacc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vb, pb.v, oacc[f], 0, 0, 0);
        }
      };

      // two register sets: the keys and values of pair pr+1 travel while pair pr is processed
      KV ra, rb;
      load_pair(ra, 0);
      int pr = 0;
      bool done = false;
      while (pr + 1 < npairs) {
        load_pair(rb, pr + 1);
        __builtin_amdgcn_sched_barrier(0);
        process(ra, pr);
        ++pr;
        if (pr + 1 >= npairs) {
          process(rb, pr);
          done = true;
          break;
        }
        load_pair(ra, pr + 1);
        __builtin_amdgcn_sched_barrier(0);
        process(rb, pr);
        ++pr;
      }
      if (!done) process(ra, pr);
    }

    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int f = 0; f < NVF; ++f) {
      oacc[f][0] *= vnorm_inv; oacc[f][1] *= vnorm_inv; oacc[f][2] *= vnorm_inv; oacc[f][3] *= vnorm_inv;
    }

    const int S = x - p;                // list position of this (b, j) sequence's first pair
    const int first_w = S / C;
    const int nrec = (S + P - 1) / C - first_w + 1;
    if (nrec == 1) {
      // this segment is the whole sequence: normalise and emit the packed O-projection operand directly
      if (n < G) {
        const float inv = 1.f / l_run;
#pragma unroll
        for (int f = 0; f < NVF; ++f) {
          union { uint16_t s[4]; u32x2 v; } hi, lo;
#pragma unroll
          for (int i = 0; i < 4; ++i) split_f16(oacc[f][i] * inv, hi.s[i], lo.s[i]);
          const int k = (j * G + n) * HD + f * 16 + g * 4;
          *reinterpret_cast<u32x2*>(xo + attn_out_offset(k, b, 0, MT, first_row, Hq * HD / 16)) = hi.v;
          *reinterpret_cast<u32x2*>(xo + attn_out_offset(k, b, 1, MT, first_row, Hq * HD / 16)) = lo.v;
        }
      }
    } else {
      // park the record [2w | 2w + 1][head n][o(HD), m, l]; a separate small kernel merges the records (a kernel
      // boundary is a far cheaper hand-over here than in-kernel device-scope signalling)
      float* rec = part + (int64_t)(2 * w + (x == w * C ? 0 : 1)) * G * PSTRIDE;
      if (n < G) {
#pragma unroll
        for (int f = 0; f < NVF; ++f)
          *reinterpret_cast<float4*>(rec + n * PSTRIDE + f * 16 + g * 4) = make_float4(oacc[f][0], oacc[f][1], oacc[f][2], oacc[f][3]);
        if (g == 0) {
          rec[n * PSTRIDE + HD] = m_run;
          rec[n * PSTRIDE + HD + 1] = l_run;
        }
      }
    }
    x += np;
    remaining -= np;
    p = 0;
    if (++j == Hkv) {
      j = 0;
      if (++b < batch && remaining > 0) ctx = __builtin_amdgcn_readfirstlane(seq_lens[b]);
    }
  }
}

// Merges the records of one (sequence, kv head) and writes the packed hi/lo operand of the O projection.  The records are cut into eight runs, in
// key order; a run is added up record by record, then the runs one by one, so the order of all sums depends on the number of records alone: sums
// split by the query heads that share a kv head moved the cache entries of a chunk's last position in their last bits, and with them, after 32
// layers, a chunked prompt's logits by 2e-4.  A wavefront takes runs of one query head, two (four with 64-wide heads) side by side: 16-byte loads,
// up to eight records of each run on their way.  Up to eight records are runs of one: the threads that write the result read them all, without LDS
// (eight query heads, 33 and 128 sequences 5.5 -> 5.0, 5.6 -> 5.1 us).  Sequences that were a single segment were finished by the attention kernel.
// Bound by the launch, memory round trips (plan, records), a compute unit's intake and instruction fetch.  Against a wavefront per run for all
// query heads (4-byte loads, four records on their way), eight kv heads of 128, us by query heads per kv head: one sequence of 1041 tokens, four 6.5
// -> 5.3; of 2000 and 40 000, two 6.2 -> 4.8, 6.8 -> 5.2, four 7.2 -> 6.1, 8.1 -> 6.6, eight 11.2 -> 8.2, 12.3 -> 9.2; three of 4000 to 8000, four 6.0
// -> 5.1, eight 9.0 -> 6.8; 16 to 128 sequences, up to four 4.6 to 4.9 on both sides, eight 5.1 to 7.7 -> 4.8 to 5.1; heads of 64, one sequence of
// 2000, four 7.0 -> 4.6, eight 8.7 -> 6.1.
constexpr int MERGE_RUNS = 8;
template <int HD, int G>
__global__ __launch_bounds__(1024) void decode_attn_merge_kernel(const int32_t* __restrict__ seq_lens, int Hkv, const int32_t* __restrict__ hdr,
                                                                  const int32_t* __restrict__ pref, const float* __restrict__ part,
                                                                  uint16_t* __restrict__ xo, int MT, int first_row, int waves) {
  constexpr int PSTRIDE = HD + 4, LR = HD / 4, SIDE = 64 / LR, U = 8;  // lanes of a record, runs side by side, records of a run on their way
  const int j = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int C = hdr[1];
  const int P = max(0, (seq_lens[b] + 31) / 32);
  const int S = pref[b] * Hkv + j * P;  // list position of this sequence's first pair
  const int first_w = S / C;
  const int nrec = (S + P - 1) / C - first_w + 1;
  if (nrec <= 1) return;
  const int first_slot = 2 * first_w + (S == first_w * C ? 0 : 1);  // later wavefronts begin with this sequence: even records
  const int per = (nrec + MERGE_RUNS - 1) / MERGE_RUNS, n_runs = (nrec + per - 1) / per;
  float M, L;
  f32x4 o;
  // (one of the two products of a sum is rounded before it: which one is part of the order)
  auto take = [&](float mv, float lv, f32x4 ov, bool old_rounded) __attribute__((always_inline)) {
    const float Mn = fmaxf(M, mv), ref = Mn == NEG_INF ? 0.f : Mn;
    const float a = __builtin_amdgcn_exp2f(M - ref), w = __builtin_amdgcn_exp2f(mv - ref);
    L = __builtin_fmaf(L, a, lv * w);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = old_rounded ? __builtin_fmaf(ov[i], w, o[i] * a) : __builtin_fmaf(o[i], a, ov[i] * w);
    M = Mn;
  };
  auto add_run = [&](int hh, int c, int r0, int r_end, int longest, bool old_rounded) __attribute__((always_inline)) {
    M = NEG_INF;
    L = 0.f;
    o = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < longest; s0 += U) {
      f32x4 ov[U];
      float2 ml[U];
      auto request = [&](int u) __attribute__((always_inline)) {
        const int r = min(r0 + s0 + u, nrec - 1);
        const float* rec = part + ((int64_t)(r == 0 ? first_slot : 2 * (first_w + r)) * G + hh) * PSTRIDE;
        ml[u] = *reinterpret_cast<const float2*>(rec + HD);
        ov[u] = *reinterpret_cast<const f32x4*>(rec + c);
      };
      // (no more than there are: eight for two or three cost 1.2 us of a launch with 128 sequences, eight for five 0.7 with one of 33 records)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= longest) break;
        request(u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= longest) break;
        if (r0 + s0 + u < r_end) take(ml[u].x, ml[u].y, ov[u], old_rounded);
      }
    }
  };
  __shared__ float mid[MERGE_RUNS][G][PSTRIDE];
  if (per > 1) {
    const int hh = wave % G, sub = lane / LR, c = (lane % LR) * 4;
    for (int run0 = wave / G * SIDE; run0 < n_runs; run0 += waves / G * SIDE) {
      const int r0 = (run0 + sub) * per;
      add_run(hh, c, r0, min(nrec, r0 + per), per, HD == 64);
      if (run0 + sub < n_runs) {
        float* out = mid[run0 + sub][hh];
        *reinterpret_cast<f32x4*>(out + c) = o;
        if (c == 0) *reinterpret_cast<float2*>(out + HD) = make_float2(M, L);
      }
    }
    __syncthreads();
  }
  const int hh = threadIdx.x / LR, c = (threadIdx.x % LR) * 4;
  if (hh >= G) return;
  if (per > 1) {
    M = mid[0][hh][HD];
    L = mid[0][hh][HD + 1];
    o = *reinterpret_cast<const f32x4*>(&mid[0][hh][c]);
    for (int u = 1; u < n_runs; ++u) take(mid[u][hh][HD], mid[u][hh][HD + 1], *reinterpret_cast<const f32x4*>(&mid[u][hh][c]), false);
  } else {  // runs of one record
    add_run(hh, c, 0, nrec, nrec, false);
  }
  const float inv = 1.f / L;
  union { uint16_t s[4]; u32x2 v; } hi, lo;
#pragma unroll
  for (int i = 0; i < 4; ++i) split_f16(o[i] * inv, hi.s[i], lo.s[i]);
  const int k = (j * G + hh) * HD + c;
  *reinterpret_cast<u32x2*>(xo + attn_out_offset(k, b, 0, MT, first_row, Hkv * G * HD / 16)) = hi.v;
  *reinterpret_cast<u32x2*>(xo + attn_out_offset(k, b, 1, MT, first_row, Hkv * G * HD / 16)) = lo.v;
}

// ------------------------------------------------------------------------------------------------
// Greedy next token: index of the largest logit, the lowest index winning ties.  The output head's workgroups leave the largest of their rows
// per token; one workgroup per token combines these.  Two kernels that read the logits again took 9 us, 19 with 128 sequences; this one takes
// 4.2, and the head as much longer as it compares and exchanges (no shorter with the records of a workgroup side by side, which take 0.5 us more
// to read here, nor with the registers of four wavefronts per SIMD where FP8 weights and 17 to 32 tokens have those of three): head and all behind it, 4096
// columns and 128 256 rows, us, 1, 17, 32, 64 and 128 sequences 174.5 -> 173.0, 188.3 -> 187.4, 191.6 -> 191.3, 215.1 -> 210.0, 314.7 -> 315.3;
// FP8 95.8 -> 91.4, 109.2 -> 106.3, 113.9 -> 110.1, 148.8 -> 144.7, 302.3 -> 301.3.  (With one narrow layer in front, 24, 32 and 100 sequences: 253.9 ->
// 252.6, 264 -> 262.4, 389.8 -> 392.2; FP8 167.3 -> 169.3, 176.0 -> 177.7, 364.2 -> 369.6.)
__global__ __launch_bounds__(256) void argmax_kernel(const float* __restrict__ val, const int* __restrict__ idx, int n, int32_t* __restrict__ out) {
  const int tid = threadIdx.x;
  float best = NEG_INF;
  int bi = 0x7fffffff;
#pragma unroll 4
  for (int q = tid; q < n; q += 256) argmax_take(best, bi, val[(int64_t)blockIdx.x * n + q], idx[(int64_t)blockIdx.x * n + q]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) argmax_take(best, bi, __shfl_xor(best, o), __shfl_xor(bi, o));
  __shared__ float sv[4];
  __shared__ int si[4];
  if ((tid & 63) == 0) { sv[tid >> 6] = best; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w) argmax_take(best, bi, sv[w], si[w]);
    // a row without any ordered value (all NaN) has no largest element: token 0, never an index outside the vocabulary
    out[blockIdx.x] = bi == 0x7fffffff ? 0 : bi;
  }
}

// ------------------------------------------------------------------------------------------------
// Host side

// Workgroups a skinny GEMM should spread over (split-K is used when the row tiles alone are fewer): one per compute
// unit, so that no compute unit carries two of a kernel's workgroups while others carry one.  Tunable through the
// environment variable WWW_GEMM_WG_TARGET, read once.
int decode_wg_target() {
  static int v = 0;
  if (!v) {
    const char* e = getenv("WWW_GEMM_WG_TARGET");
    if (e) {
      v = atoi(e);
    } else {
      int dev = 0, cus = 0;
      if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) v = cus;
      else (void)hipGetLastError();
      if (v < 1) v = 256;
    }
    if (v < 1) v = 1;
  }
  return v;
}

int decode_MT(int batch) { return batch <= 16 ? 1 : batch <= 32 ? 2 : batch <= 64 ? 4 : ((batch + 127) / 128) * 8; }

void choose_split(int row_tiles, int zb, int KB, int* ksplit, int* kb_per_split) {
  int want = decode_wg_target() / (row_tiles * zb);
  if (want < 1) want = 1;
  if (want > MAX_KSPLIT) want = MAX_KSPLIT;
  int per = (KB + want - 1) / want;
  per = (per + 3) / 4 * 4;
  if (per < 8) per = 8;  // at least two k chunks per workgroup, so the load pipeline has something to overlap
  *kb_per_split = per;
  *ksplit = (KB + per - 1) / per;
}

// largest split factor the decode path will use for a GEMM with NRG row groups, KB k blocks and MT token groups (for
// workspace sizing)
int decode_gemm_ksplit(int NRG, int KB, int MT) {
  int most = 1;
  for (int zb = MT > 8 ? MT / 8 : 1; zb <= (MT + 3) / 4; ++zb) {  // workgroups per row tile and split, see launch_gemm
    int ks, per;
    choose_split((NRG + 7) / 8, zb, KB, &ks, &per);
    if (ks > most) most = ks;
  }
  return most;
}

// Tokens per workgroup (16 mtk), workgroups per row tile (zb) and split of the k range of skinny_gemm_kernel
struct SkinnyShape { int mtk, zb, ksplit, kb_per_split; };
static SkinnyShape skinny_shape(const www_model* m, int epi, int NRG, int KB, int M) {
  const int row_tiles = (NRG + 7) / 8, MT = decode_MT(M);
  // Above 64 tokens the two wide GEMMs may take 128 tokens per workgroup: every compute unit takes in about 55 KB per us, and
  // 128 rows x 128 tokens need 24 KB per k block where two workgroups of 64 tokens need 32 (with FP8 weights 20 and 24).
  // A round of 128 tokens on all compute units takes about 1.75 (FP8: 1.9) times as long as one of 64 (8B shape, gate/up 73
  // and 42 us), so they are taken where they save that many rounds: 8B shape, 128 sequences 7000 -> 6670 us a step, 256:
  // 11 840 -> 11 440.  Elsewhere they cost: 192 sequences 10 160 -> 10 850 us, with FP8 weights 9290 -> 10 400, 1B shape 65
  // sequences 1456 -> 1530.  The split-K GEMMs, whose epilogues then exceed the registers, are slower that way (QKV
  // 36 -> 52 us), and so are int4 weights (a step of 100 sequences 7250 -> 7700 us).  A range of k is never split there: more
  // than half of the compute units have a row tile each, or there would be no round to save.
  auto rounds = [&](int tokens) { return (float)((row_tiles * ((M + tokens - 1) / tokens) + decode_wg_target() - 1) / decode_wg_target()); };
  const bool wide = (epi == EPI_SWIGLU || epi == EPI_LOGITS) && !m->int4_group && !m->wsplit && rounds(128) * (m->fp8 ? 1.9f : 1.75f) < rounds(64);
  SkinnyShape s;
  s.mtk = MT < 8 ? MT : wide ? 8 : 4;
  s.zb = MT < 8 ? 1 : (M + 16 * s.mtk - 1) / (16 * s.mtk);  // (not MT / mtk: the last 64 tokens may all be padding)
  choose_split(row_tiles, s.zb, KB, &s.ksplit, &s.kb_per_split);
  return s;
}

// false: the shape the rules chose has no kernel, nothing was launched
template <int EPI>
static bool launch_gemm(www_model* m, GemmP& p, const SmallShape& small, hipStream_t st, const MidShape& mid = {0, 0, 0}) {
  if (small.R) return launch_small_gemm<EPI>(m, p, small, st);
  if (mid.R) return launch_mid_gemm(m, p, mid, st);
  bool launched = false;
  constexpr bool wide_epi = EPI == EPI_SWIGLU || EPI == EPI_LOGITS;
  const SkinnyShape s = skinny_shape(m, EPI, p.NRG, p.KB, p.M);
  const int mtk = s.mtk, zb = s.zb;
  p.ksplit = s.ksplit;
  p.kb_per_split = s.kb_per_split;
  p.MT = decode_MT(p.M);
  p.partial = m->partial;
  p.counters = m->counters;
  p.fault_flag = m->fault_dev;
  p.row_tiles = (p.NRG + 7) / 8;
  p.zbs = zb;
  p.fence_handover = m->handover_fence;
  if (p.wfactor == 0.f) p.wfactor = 1.f;  // not set: an unscaled matrix
  dim3 grid(8 * ((p.row_tiles + 7) / 8) * p.ksplit * zb);
#define LAUNCH(MTK_, WM_, KH_) { hipLaunchKernelGGL((skinny_gemm_kernel<MTK_, WM_, EPI, KH_>), grid, dim3(256 * KH_), 0, st, p); launched = true; }
#define LAUNCH2(WM_, KH_) { if constexpr (wide_epi || WM_ != WMODE_INT4) LAUNCH(2, WM_, KH_) }  // (int4, narrow: small_gemm_kernel)
#define LAUNCH8(WM_) { if constexpr (wide_epi) LAUNCH(8, WM_, 2) }
  // With more than 32 tokens the MFMAs of a chunk take a third of a wavefront's time; in the gate/up GEMM (no split-K,
  // 32 chunks per workgroup) two wavefronts per SIMD (KH = 2) hide them behind each other's waits: 53 -> 49.5 us at 64
  // tokens of the 8B shape.  The split-K GEMMs walk 4 - 14 chunks and are bound by their fixed costs; the hand-over
  // between the wavefront halves costs them as much as it saves, so they stay at KH = 1.
  constexpr int kh4 = EPI == EPI_SWIGLU ? 2 : 1;
  if (m->int4_group) {
    // unpacking the codes takes longer than the weight stream, so from 17 tokens on two wavefronts per SIMD share it (8B shape,
    // gate/up at 30 tokens 31.8 -> 29.8 us, at 60 47.7 -> 42.4; QKV and the residual GEMMs 1 - 3 us at 60 - 100).  Not with up to
    // 16 tokens (each chunk is then over before the next has arrived: 23.8 -> 31.0 us), not in the output head (145 -> 166)
    // and not in the gate/up GEMM with two token groups side by side (70 -> 80)
    constexpr int ki = EPI == EPI_LOGITS ? 1 : 2;
    if (mtk == 1) LAUNCH(1, WMODE_INT4, 1)
    else if (mtk == 2) LAUNCH2(WMODE_INT4, ki)
    else if (EPI == EPI_SWIGLU && zb > 1) LAUNCH(4, WMODE_INT4, 1)
    else LAUNCH(4, WMODE_INT4, ki)
  } else if (m->fp8) {
    if (mtk == 1) LAUNCH(1, WMODE_FP8, 1) else if (mtk == 2) LAUNCH2(WMODE_FP8, 1) else if (mtk == 4) LAUNCH(4, WMODE_FP8, kh4) else LAUNCH8(WMODE_FP8)
  } else if (m->wsplit) {
    if (mtk == 1) LAUNCH(1, WMODE_SPLIT, 1) else if (mtk == 2) LAUNCH2(WMODE_SPLIT, 1) else LAUNCH(4, WMODE_SPLIT, 1)
  } else {
    if (mtk == 1) LAUNCH(1, WMODE_F16, 1) else if (mtk == 2) LAUNCH2(WMODE_F16, 1) else if (mtk == 4) LAUNCH(4, WMODE_F16, kh4) else LAUNCH8(WMODE_F16)
  }
#undef LAUNCH2
#undef LAUNCH8
#undef LAUNCH
  return launched;
}

// Kernel (0: skinny_gemm_kernel, 1: small_gemm_kernel, 4: mid_gemm_kernel), tokens and rows per workgroup and k splits of GEMM `which`
// (0 QKV, 1 O, 2 gate/up, 3 down, 4 output head) of a decode step; false: there is no such kernel
bool decode_route(const www_model* m, int which, int batch, int32_t out[4]) {
  const int epi[5] = {EPI_QKV, EPI_RESID, EPI_SWIGLU, EPI_RESID, EPI_LOGITS};
  const int NRG = (which == 0 ? m->QKVN : which == 2 ? 2 * m->F : which == 4 ? m->V : m->d) / 16;
  const int KB = (which == 1 ? m->QD : which == 3 ? m->Fp : m->d) / 32;
  if (const SmallShape s = small_gemm_route(m, epi[which], NRG, KB, batch); s.R) {
    out[0] = 1; out[1] = s.xf == 1 ? 8 : s.xf == 2 ? 16 : 32; out[2] = 16 * s.R * s.RW; out[3] = s.ks;
    return small_gemm_built(m, epi[which], s);
  } else if (const MidShape g = mid_gemm_route(m, epi[which], NRG, KB, batch); g.R) {
    out[0] = 4; out[1] = 64; out[2] = 16 * g.R; out[3] = g.ks;
    return mid_gemm_built(m, g);
  } else {
    const SkinnyShape k = skinny_shape(m, epi[which], NRG, KB, batch);
    out[0] = 0; out[1] = 16 * k.mtk; out[2] = GEMM_TILE_ROWS; out[3] = k.ksplit;
    return k.mtk != 2 || !m->int4_group || which == 2 || which == 4;  // (narrow int4 products of 17 to 32 tokens: the other kernel)
  }
}

// wavefronts the decode attention kernel keeps resident on the whole device (its grid), a multiple of 4
int decode_attn_resident_waves(int hd, int G) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 1024;
  }
  hipError_t e = hipErrorInvalidValue;
#define OCC(HD_, G_) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_attn_kernel<HD_, G_>, 256, 0)
  if (hd == 128) {
    if (G == 1) OCC(128, 1); else if (G == 2) OCC(128, 2); else if (G == 4) OCC(128, 4); else OCC(128, 8);
  } else {
    if (G == 1) OCC(64, 1); else if (G == 2) OCC(64, 2); else if (G == 4) OCC(64, 4); else OCC(64, 8);
  }
#undef OCC
  if (e != hipSuccess || per_cu < 1) { (void)hipGetLastError(); per_cu = 1; }
  return per_cu * cus * 4;
}

// Placement probe: every workgroup records the id of the XCD it runs on.
__global__ __launch_bounds__(256) void xcc_probe_kernel(int32_t* __restrict__ out) {
  const int xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15;  // HW_REG_XCC_ID, bits 3:0
  if (threadIdx.x == 0) out[blockIdx.x] = xcc;
}

// 1 if workgroups whose ids are equal modulo 8 were all placed on the same XCD in a probe launch of n workgroups
// (scratch_dev: n ints of device memory), 0 if not, -1 on a HIP error.
int decode_probe_placement(int32_t* scratch_dev, int n, hipStream_t st) {
  std::vector<int32_t> h(n);
  hipLaunchKernelGGL(xcc_probe_kernel, dim3(n), dim3(256), 0, st, scratch_dev);
  if (hipMemcpyAsync(h.data(), scratch_dev, (size_t)n * 4, hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
  if (hipStreamSynchronize(st) != hipSuccess) return -1;
  for (int i = 8; i < n; ++i)
    if (h[i] != h[i & 7]) return 0;
  return 1;
}

static AttnPlan plan_of(const www_model* m, const int32_t* lens, int batch) {
  return {lens, batch, m->Hkv, m->attn_waves, m->attn_hdr, m->attn_start, m->attn_pref};
}
static size_t plan_lds_bytes(int batch) { return batch + 2 < 256 ? 1024 : (size_t)(batch + 2) * 4; }
void launch_attn_plan(www_model* m, const int32_t* lens, int batch, hipStream_t st) {
  hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(256), plan_lds_bytes(batch), st, plan_of(m, lens, batch));
}

void launch_decode_attn(www_model* m, int l, const int32_t* lens, const int32_t* table, int batch, uint16_t* out, int MT, int first_row, hipStream_t st) {
  const uint16_t *kplane = m->kv + (int64_t)(2 * l) * m->kv_plane, *vplane = m->kv + (int64_t)(2 * l + 1) * m->kv_plane;
  const float* kvscale = m->kv_scales + (int64_t)l * m->kv_scale_plane;
  // all eight runs of a head side by side where a wavefront takes no more than one query head's at a time and every workgroup has a compute unit (8B
  // shape, a layer of a step, us: one sequence of 2000 tokens 34.8 -> 34.2, 16 47.3 -> 47.0; 64 72.1 -> 72.9, 128 80.3 -> 82.3)
  const int merge_waves = m->G * m->hd > 256 && m->Hkv * batch <= decode_wg_target() ? 16 : 8;
#define ATTN(HD_, G_)                                                                                                              \
  {                                                                                                                                \
    hipLaunchKernelGGL((decode_attn_kernel<HD_, G_>), dim3(m->attn_waves / 4), dim3(256), 0, st, m->q_hi, m->q_lo, kplane, vplane,  \
                       kvscale, lens, table, batch, (int)m->cfg.max_blocks_per_seq, m->Hq, m->Hkv, m->attn_hdr, m->attn_start,      \
                       m->attn_part, out, MT, first_row);                                                                           \
    hipLaunchKernelGGL((decode_attn_merge_kernel<HD_, G_>), dim3(m->Hkv, batch), dim3(64 * merge_waves), 0, st, lens, m->Hkv,               \
                       m->attn_hdr, m->attn_pref, m->attn_part, out, MT, first_row, merge_waves);                                   \
  }
  if (m->hd == 128) {
    if (m->G == 1) ATTN(128, 1) else if (m->G == 2) ATTN(128, 2) else if (m->G == 4) ATTN(128, 4) else ATTN(128, 8)
  } else {
    if (m->G == 1) ATTN(64, 1) else if (m->G == 2) ATTN(64, 2) else if (m->G == 4) ATTN(64, 4) else ATTN(64, 8)
  }
#undef ATTN
}

int run_decode(www_model* m, const int32_t* tok, const int32_t* lens, const int32_t* table, int batch, float* logits, int32_t* next,
               bool from_last_qkv, hipStream_t st) {
  const int MT = decode_MT(batch);
  const int d = m->d;
  float* const ssq = MT <= 2 ? m->ssq_rows : m->ssq;
  if (!from_last_qkv) {
    prof_mark(m, PK_EMBED, st);
    if (m->cfg.weight_dtype == WWW_DTYPE_F32)
      hipLaunchKernelGGL(embed_pack_kernel<float>, dim3(batch + 1), dim3(256), plan_lds_bytes(batch), st, tok, (const float*)m->embed, d, m->layers[0].attn_norm,
                         m->h, ssq, (uint16_t*)m->xq, MT, plan_of(m, lens, batch));
    else
      hipLaunchKernelGGL(embed_pack_kernel<uint16_t>, dim3(batch + 1), dim3(256), plan_lds_bytes(batch), st, tok, (const uint16_t*)m->embed, d,
                         m->layers[0].attn_norm, m->h, ssq, (uint16_t*)m->xq, MT, plan_of(m, lens, batch));
  }
  bool launched = true;
  int n_ssq = 1;  // entries per token of the sum-of-squares table: one per row group or per row tile of the GEMM that wrote it
  auto resid_entries = [&](const SmallShape& s, const MidShape& g) { const int rg = s.R ? 1 : g.R ? g.R : 8; return (d / 16 + rg - 1) / rg; };
  // the same in every layer
  const SmallShape s_qkv = small_gemm_route(m, EPI_QKV, m->QKVN / 16, d / 32, batch), s_o = small_gemm_route(m, EPI_RESID, d / 16, m->QD / 32, batch);
  const SmallShape s_gu = small_gemm_route(m, EPI_SWIGLU, 2 * m->F / 16, d / 32, batch), s_down = small_gemm_route(m, EPI_RESID, d / 16, m->Fp / 32, batch);
  const MidShape m_o = mid_gemm_route(m, EPI_RESID, d / 16, m->QD / 32, batch), m_down = mid_gemm_route(m, EPI_RESID, d / 16, m->Fp / 32, batch);
  const float qscale = 1.4426950408889634f / sqrtf((float)m->hd);
  for (int l = from_last_qkv ? m->L - 1 : 0; l < m->L; ++l) {
    const LayerW& w = m->layers[l];
    uint16_t* kplane = (uint16_t*)m->kv + (int64_t)(2 * l) * m->kv_plane;
    uint16_t* vplane = (uint16_t*)m->kv + (int64_t)(2 * l + 1) * m->kv_plane;
    float* kvscale = m->kv_scales + (int64_t)l * m->kv_scale_plane;
    if (!from_last_qkv) {
      GemmP p = {};
      p.W = (const u32x4*)(w.wqkv8 ? (const void*)w.wqkv8 : (const void*)w.wqkv); p.Wlo = (const u32x4*)w.wqkv_lo; p.wfactor = w.sqkv; p.Wscale = (const u32x2*)w.gqkv;
      p.NRG = m->QKVN / 16; p.KB = d / 32;
      p.X = (const u32x4*)m->xq; p.M = batch;
      p.ssq_in = ssq; p.n_ssq_in = n_ssq; p.inv_dim = 1.f / d; p.eps = m->cfg.rms_eps;
      p.q_hi = m->q_hi; p.q_lo = m->q_lo; p.qscale = qscale; p.kplane = kplane; p.vplane = vplane; p.kvscale = kvscale; p.seq_lens = lens; p.table = table; p.mbs = m->cfg.max_blocks_per_seq;
      p.hd = m->hd; p.Hq = m->Hq; p.Hkv = m->Hkv; p.rope = m->rope; p.qk_gain = w.qk_gain;
      prof_mark(m, PK_QKV, st);
      launched &= launch_gemm<EPI_QKV>(m, p, s_qkv, st);
    }
    prof_mark(m, PK_ATTN, st);
    launch_decode_attn(m, l, lens, table, batch, (uint16_t*)m->xo, MT, -1, st);
    {
      GemmP p = {};
      p.W = (const u32x4*)(w.wo8 ? (const void*)w.wo8 : (const void*)w.wo); p.Wlo = (const u32x4*)w.wo_lo; p.wfactor = w.so; p.Wscale = (const u32x2*)w.go;
      p.NRG = d / 16; p.KB = m->QD / 32;
      p.X = (const u32x4*)m->xo; p.M = batch;
      p.h = m->h; p.gain_next = w.ffn_norm; p.xnext = (uint16_t*)m->xq; p.ssq_out = ssq; p.d = d;
      prof_mark(m, PK_OPROJ, st);
      launched &= launch_gemm<EPI_RESID>(m, p, s_o, st, m_o);
      n_ssq = resid_entries(s_o, m_o);
    }
    {
      GemmP p = {};
      p.W = (const u32x4*)(w.wgu8 ? (const void*)w.wgu8 : (const void*)w.wgu); p.Wlo = (const u32x4*)w.wgu_lo; p.wfactor = w.sgu; p.Wscale = (const u32x2*)w.ggu;
      p.NRG = 2 * m->F / 16; p.KB = d / 32;
      p.X = (const u32x4*)m->xq; p.M = batch;
      p.ssq_in = ssq; p.n_ssq_in = n_ssq; p.inv_dim = 1.f / d; p.eps = m->cfg.rms_eps;
      p.xa = (uint16_t*)m->xa; p.F = m->F;
      prof_mark(m, PK_GATEUP, st);
      launched &= launch_gemm<EPI_SWIGLU>(m, p, s_gu, st);
    }
    {
      GemmP p = {};
      p.W = (const u32x4*)(w.wd8 ? (const void*)w.wd8 : (const void*)w.wd); p.Wlo = (const u32x4*)w.wd_lo; p.wfactor = w.sd; p.Wscale = (const u32x2*)w.gd;
      p.NRG = d / 16; p.KB = m->Fp / 32;
      p.X = (const u32x4*)m->xa; p.M = batch;
      p.h = m->h; p.gain_next = (l + 1 < m->L) ? m->layers[l + 1].attn_norm : m->final_norm;
      p.xnext = (uint16_t*)m->xq; p.ssq_out = ssq; p.d = d;
      prof_mark(m, PK_DOWN, st);
      launched &= launch_gemm<EPI_RESID>(m, p, s_down, st, m_down);
      n_ssq = resid_entries(s_down, m_down);
    }
  }
  float* lg = logits ? logits : m->logits_buf;
  {
    GemmP p = {};
    p.W = (const u32x4*)(m->lm_head8 ? (const void*)m->lm_head8 : (const void*)m->lm_head); p.Wlo = (const u32x4*)m->lm_head_lo; p.wfactor = m->s_lm; p.Wscale = (const u32x2*)m->g_lm;
    p.NRG = m->V / 16; p.KB = d / 32;
    p.X = (const u32x4*)m->xq; p.M = batch;
    p.ssq_in = ssq; p.n_ssq_in = n_ssq; p.inv_dim = 1.f / d; p.eps = m->cfg.rms_eps;
    p.logits = lg; p.V = m->V;
    prof_mark(m, PK_LMHEAD, st);
    if (next) { p.best_val = m->argmax_val; p.best_idx = m->argmax_idx; }
    launched &= launch_gemm<EPI_LOGITS>(m, p, small_gemm_route(m, EPI_LOGITS, m->V / 16, d / 32, batch), st);
    if (next) {
      prof_mark(m, PK_ARGMAX, st);
      hipLaunchKernelGGL(argmax_kernel, dim3(batch), dim3(256), 0, st, m->argmax_val, m->argmax_idx, p.row_tiles, next);
    }
  }
  prof_mark(m, -1, st);
  if (!launched) {
    set_error("decode: no kernel for the shape chosen for a GEMM");
    return WWW_E_HIP;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("decode launch failed: %s", hipGetErrorString(e));
    return WWW_E_HIP;
  }
  return WWW_OK;
}
