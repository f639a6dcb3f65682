// Prefill path (many new tokens per sequence): ragged-batch bookkeeping, embedding, RMSNorm,
// LDS-tiled fp16 MFMA GEMM with rotary + KV-cache write / residual / SwiGLU epilogues, and causal
// paged flash attention over cached prefix + new tokens.  This pass fills the KV cache; the logits
// come from each sequence's last position, whose activations are kept in hi/lo precision: either the whole
// position runs through the decode path afterwards, or it rides along as rows of its own (below).
#include <type_traits>

#include "common.h"

#define NEG_INF (-__builtin_inff())

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

#define ATTN_TQ 64  // query rows per attention workgroup

// Last positions as rows of a prefill call.  The decode pass that follows a prefill reads every weight a second time (8B shape, one
// sequence: 3.3 of the 11 ms of a 333-token prompt).  Where the rows cost the GEMMs less than that pass (prefill_rides), the
// last position of sequence s travels through all layers but the rest of the last one as two more rows of the same GEMMs:
// the hi parts of its activations are row first_last + 32 (s / 16) + s % 16, the lo parts 16 rows behind, so both are columns
// of one 32-token group and a lane finds the other part 16 lanes away.  The epilogues add the two products and write the
// residual (fp32, m->h), hi and lo operands, queries and cache codes that the decode path's kernels would have written; the
// ordinary row of that position still runs along, but leaves the cache alone.  Attention at those positions is the
// decode path's kernel in every layer, and that path takes over behind the last layer's QKV product.
__host__ __device__ __forceinline__ int last_row_of(int first_last, int s) { return first_last + (s >> 4) * 32 + (s & 15); }

// ------------------------------------------------------------------------------------------------
// Ragged batch bookkeeping (one workgroup).  meta[0] = number of attention tiles.
__global__ __launch_bounds__(1024) void prefill_meta_kernel(const int32_t* __restrict__ tokens, const int32_t* __restrict__ q_lens,
                                                             const int32_t* __restrict__ seq_lens, int batch, int T,
                                                             int32_t* __restrict__ row_seq, int32_t* __restrict__ row_pos,
                                                             int32_t* __restrict__ tile_seq, int32_t* __restrict__ tile_q0,
                                                             int32_t* __restrict__ meta, int32_t* __restrict__ last_tok,
                                                             int32_t* __restrict__ cum /* [2*(batch+1)] scratch */,
                                                             int first_last, int rows /* 0, T: the last positions do not ride along */) {
  int32_t* cum_rows = cum;
  int32_t* cum_tiles = cum + batch + 1;
  if (threadIdx.x == 0) {
    int r = 0, tl = 0;
    for (int b = 0; b < batch; ++b) {
      cum_rows[b] = r;
      cum_tiles[b] = tl;
      r += q_lens[b];
      tl += (q_lens[b] + ATTN_TQ - 1) / ATTN_TQ;
    }
    cum_rows[batch] = r;
    cum_tiles[batch] = tl;
    meta[0] = tl;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < T; r += blockDim.x) {
    int lo = 0, hi = batch - 1;  // last b with cum_rows[b] <= r
    while (lo < hi) {
      int mid = (lo + hi + 1) >> 1;
      if (cum_rows[mid] <= r) lo = mid; else hi = mid - 1;
    }
    // (the sign marks an ordinary row whose cache entry is written by the rows of its last position)
    row_seq[r] = first_last && r == cum_rows[lo + 1] - 1 ? lo | (int)0x80000000 : lo;
    row_pos[r] = seq_lens[lo] - q_lens[lo] + (r - cum_rows[lo]);
  }
  for (int r = T + threadIdx.x; r < rows; r += blockDim.x) {  // padding, then the rows of the last positions
    const int s = r < first_last ? 0 : min(((r - first_last) >> 5) * 16 + (r & 15), batch - 1);
    row_seq[r] = s;
    row_pos[r] = seq_lens[s] - 1;
  }
  for (int b = threadIdx.x; b < batch; b += blockDim.x) {
    int nt = cum_tiles[b + 1] - cum_tiles[b];
    for (int i = 0; i < nt; ++i) {
      tile_seq[cum_tiles[b] + i] = b;
      tile_q0[cum_tiles[b] + i] = i * ATTN_TQ;
    }
    last_tok[b] = tokens[cum_rows[b + 1] - 1];
  }
}

// The residual stream of the prefill path is only ever touched by the embedding kernel and by the residual epilogues of
// the O and down projections, which both tile it 256 tokens x 256 rows with the same accumulator layout.  It is
// therefore kept in that layout ("register image"): block (token tile tt, row tile rt) holds 64 Ki floats ordered
// [wavefront wn*2+wt][rb][tb][q4][lane][4], element = the lane's four consecutive rows
//   row   = rt*256 + wn*128 + rb*32 + q4*8 + (lane/32)*4 + e,   token = tt*256 + wt*128 + tb*32 + lane%32,
// so that every load and store of an epilogue is one contiguous KiB per wavefront instead of 64 pieces of 16 bytes
// that lie a whole token row apart.
__device__ __forceinline__ int64_t hp_image_offset(int tt, int rt, int n_rt, int wave, int rb, int tb, int q4, int lane) {
  return (((((((int64_t)tt * n_rt + rt) * 4 + wave) * 4 + rb) * 4 + tb) * 4 + q4) * 64 + lane) * 4;
}
// the same for token t and row n (a multiple of 4)
__device__ __forceinline__ int64_t hp_image_offset_of(int64_t t, int n, int n_rt) {
  const int w256 = (int)(t & 255), c = n & 255;
  const int wave = (c >> 7) * 2 + (w256 >> 7), rb = (c & 127) >> 5, tb = (w256 & 127) >> 5, q4 = (c & 31) >> 3;
  const int lane = ((c & 7) >> 2) * 32 + (w256 & 31);
  return hp_image_offset((int)(t >> 8), n >> 8, n_rt, wave, rb, tb, q4, lane);
}

// Embedding rows: residual stream h = E[token] (fp32), the first GEMM operand fp16(h * gain) in the packed prefill
// layout, and the row's sum of squares.  RMSNorm's 1/rms factor is applied by the consuming GEMM's epilogue.
// Workgroups past the T tokens: the last position of a sequence, residual row in h_last and operands hi and lo.
template <typename ET>
__global__ __launch_bounds__(256) void embed_rows_kernel(const int32_t* __restrict__ tokens, const ET* __restrict__ embed, int d,
                                                          const float* __restrict__ gain, float* __restrict__ hp,
                                                          uint16_t* __restrict__ xn, float* __restrict__ ssq, int T, int first_last,
                                                          const int32_t* __restrict__ last_tok, float* __restrict__ h_last) {
  const bool last = (int)blockIdx.x >= T;
  const int seq = (int)blockIdx.x - T;
  const int64_t r = last ? last_row_of(first_last, seq) : (int)blockIdx.x;
  const ET* row = embed + (int64_t)(last ? last_tok[seq] : tokens[r]) * d;
  float local = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {
    union { uint16_t s[4]; u32x2 v; } o, lo;
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (sizeof(ET) == 4) x[e] = (float)row[k + e];
      else x[e] = bf16_bits_to_float(((const uint16_t*)row)[k + e]);
      local += x[e] * x[e];
      split_f16(x[e] * gain[k + e], o.s[e], lo.s[e]);
    }
    float* h = last ? h_last + (int64_t)seq * d + k : hp + hp_image_offset_of(r, k, (d + 255) >> 8);
    *reinterpret_cast<float4*>(h) = make_float4(x[0], x[1], x[2], x[3]);
    *reinterpret_cast<u32x2*>(xn + packed_p_offset(r, k, d >> 4)) = o.v;
    if (last) *reinterpret_cast<u32x2*>(xn + packed_p_offset(r + 16, k, d >> 4)) = lo.v;
  }
  __shared__ float red[256];
  red[threadIdx.x] = local;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) ssq[(int64_t)r * PSSQ] = red[0];  // row r of the [token][PSSQ] table, one entry in use
  if (threadIdx.x == 0 && last) ssq[(int64_t)(r + 16) * PSSQ] = red[0];
}

// ------------------------------------------------------------------------------------------------
// Tiled GEMM  Y^T[n][t] = sum_k W[n][k] X[t][k]:  256 weight rows x 256 tokens per workgroup, four
// wavefronts each owning 128 x 128 as 4 x 4 MFMA 32x32x16 tiles.  Both operands arrive already in MFMA
// fragment order (packed weights, packed activations), so a K step of 32 is a straight 32 KiB copy into
// LDS (16 weight fragments + 16 activation fragments) and every LDS read is a conflict-free 16-byte read.
enum { PEPI_QKV = 0, PEPI_RESID = 1, PEPI_SWIGLU = 2 };
#define PGEMM_NB 4  // stage buffers of the prefill GEMM (32 KiB each)
#define PGEMM_LDS_BYTES (PGEMM_NB * 2048 * 16)
#define PGEMM_LAST_LDS_BYTES ((128 + 16 * 512) * 16)  // with last positions: sums of squares and 16 parked groups behind the loop

struct PGemmP {
  const u32x4* W;  // packed weights
  float wfactor;   // scale of the matrix (FP8 weight-only sources; 1 otherwise), applied to the result
  int NRG, KB;
  const u32x4* X;  // packed activations
  int T;           // rows of X
  int n_tt, n_rt;  // token tiles, row tiles of 256 x 256
  // last positions that ride along (kernels with LAST): ordinary tokens, first row of the last positions, their number, their
  // residual rows and (QKV) queries
  int T_new, first_last, n_last;
  float* h_last;
  uint16_t *q_hi, *q_lo;
  float qscale;
  // QKV epilogue
  const float* qk_gain;  // models with normalised query / key heads: [2][hd] gains in packed row order; null otherwise
  uint16_t* qp;
  uint16_t *kplane, *vplane;  // this layer's key / value planes of the pool (16-bit codes)
  float* kvscale;             // and its plane of scales
  const int32_t *row_seq, *row_pos, *table;
  int mbs, hd, Hq, Hkv;
  const float2* rope;
  // RMSNorm scale of the input rows (QKV and SwiGLU GEMMs): rsqrt(sum_i ssq_in[i][t] / dim + eps) multiplies the result
  const float* ssq_in;
  int n_ssq_in;
  float inv_dim, eps;
  // residual epilogue: h += result; also emits the next GEMM's operand fp16(h * gain_next) and partial sums of squares
  float* hp;
  int d;
  const float* gain_next;
  uint16_t* xn_out;
  float* ssq_out;
  // SwiGLU epilogue
  uint16_t* ap;
  int Fp;
  // the kernel of smaller tiles: its tile counts, splits of the k range, and their hand-over (as in the decode GEMMs)
  int n_ttS, n_rt128, ksplit, kb_per_split;
  float* partial;
  unsigned long long* counters;
  int fence_handover;
  int* fault_flag;
};

// Workgroup id -> tile of the prefill GEMM.  Workgroup ids are dealt round-robin to the 8 XCDs and dispatched in order,
// so a round of 256 workgroups gives every XCD 32 consecutive local indices.  Token tiles are taken in super-groups of
// 8 x GT: XCD x owns GT of them and walks the row tiles 8 at a time (32 workgroups = GT token tiles x 8 row tiles: its
// L2 sees GT + 8 operand panels per round), and all XCDs walk the row tiles in step, so a weight panel is fetched from
// memory once per super-group and found in the memory-side cache by the other seven.  The token tiles that do not
// fill a super-group follow in groups of GT with the ids' order simply transposed over the XCDs.  The map is a
// bijection from [0, n_tt * n_rt) onto the tiles (checked on the host for many shapes through www_debug_prefill_tile).
__host__ __device__ __forceinline__ void pgemm_tile_of(int id, int n_tt, int n_rt, int* tt_out, int* rt_out) {
  constexpr int GT = 4;
  const int total = n_tt * n_rt;
  const int n_sg = n_tt / (8 * GT);            // full super-groups
  const int total_sg = n_sg * 8 * GT * n_rt;   // tiles in them (a multiple of 8)
  if (id < total_sg) {
    const int x = id & 7, li = id >> 3;
    const int per_sg = GT * n_rt;              // tiles of one XCD in one super-group
    const int sg = li / per_sg, within = li % per_sg;
    *tt_out = (sg * 8 + x) * GT + within % GT;
    *rt_out = within / GT;
  } else {
    int v = id - total_sg;
    const int rest = total - total_sg, tt0 = n_sg * 8 * GT;
    if (rest % 8 == 0) v = (v % 8) * (rest / 8) + v / 8;
    const int per_group = GT * n_rt;
    const int group = v / per_group, first_tt = tt0 + group * GT;
    const int left = n_tt - first_tt;
    const int gsz = left < GT ? left : GT;
    *tt_out = first_tt + (v % per_group) % gsz;
    *rt_out = (v % per_group) / gsz;
  }
}

// Epilogue of the prefill GEMMs for TB groups of 32 tokens of one wavefront: its 128 rows are row half wn, its tokens the
// groups tb0 .. tb0 + TB - 1 of token half wt of the 256 x 256 tile (tt, rt).
//   acc[rb][tb][i] = Y^T[row][token]: row = (rg_w + rb*2)*16 + (i/4)*8 + (lane/32)*4 + i%4, token = t_w + tb*32 + lane%32
// sum_out(tb, s) receives the sum of squares of a token's new residual over the wavefront's rows (residual epilogue).
// LAST: the call's last token groups hold last positions; they are left to last_epilogue, what is computed of them here is dropped.
template <int EPI, bool QKN, int TB, bool LAST, typename SUM>
__device__ __forceinline__ void pgemm_epilogue(const PGemmP& p, f32x16 (&acc)[4][TB], int tt, int rt, int wn, int wt, int tb0, SUM sum_out) {
  const int lane = threadIdx.x & 63, wave = wn * 2 + wt;  // (position of the wavefront's rows and tokens in the 256 x 256 tile)
  const int rg_w = rt * 16 + wn * 8, t_w = tt * 256 + wt * 128 + tb0 * 32;
  const int hsel = lane >> 5;
  // the residual stream's image, whose blocks are 256 tokens: three groups of 32 may cross into the next half or block
  auto image = [&](int tb, int rb, int q4) __attribute__((always_inline)) {
    if constexpr (TB == 3) {
      const int g = tt * 8 + wt * 4 + tb0 + tb;
      return hp_image_offset(g >> 3, rt, p.n_rt, wn * 2 + ((g >> 2) & 1), rb, g & 3, q4, lane);
    } else {
      return hp_image_offset(tt, rt, p.n_rt, wave, rb, tb0 + tb, q4, lane);
    }
  };
  // Everything the epilogue needs from memory per token is requested up front for all token groups (one memory
  // round trip, two for the KV block ids), and the per-element operands of a token group (residual rows, rotary
  // factors) in one batch per group: a wavefront has no partner on its SIMD to hide a chain of dependent loads behind.
  // Addresses of tokens past the end are clamped; their results are dropped.
  int tcl[TB];
  bool tok_ok[TB];
  float scale[TB];
  int pos[TB], blk[TB];
  bool keep_cache[TB];  // (LAST) ordinary row of a last position
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int t = t_w + tb * 32 + (lane & 31);
    tok_ok[tb] = t < (LAST ? p.T_new : p.T);
    tcl[tb] = min(t, p.T - 1);
    scale[tb] = p.wfactor;
    pos[tb] = 0;
    blk[tb] = 0;
    keep_cache[tb] = false;
  }
  if constexpr (EPI != PEPI_RESID) {
    if constexpr (EPI == PEPI_QKV) {
      int seq[TB];
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        pos[tb] = p.row_pos[tcl[tb]];
        seq[tb] = p.row_seq[tcl[tb]];
        if constexpr (LAST) {
          keep_cache[tb] = seq[tb] < 0;
          seq[tb] &= 0x7fffffff;
        }
      }
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) blk[tb] = kv_block_id(p.table + (int64_t)seq[tb] * p.mbs, pos[tb]);
    }
    // the tokens' rows of the sum-of-squares table, [token][PSSQ], two token groups and 32 entries at a time (64
    // registers); entries past n_ssq_in are masked, the rest is added in tile order
    constexpr int TH = TB % 2 ? 1 : 2;
#pragma unroll
    for (int t0 = 0; t0 < TB; t0 += TH) {
      if (!p.ssq_in) break;  // no normalisation requested: the scales stay 1
      float ss[TH];
#pragma unroll
      for (int u = 0; u < TH; ++u) ss[u] = 0.f;
      for (int e0 = 0; e0 < p.n_ssq_in; e0 += 32) {
        f32x4 sq[TH][8];
#pragma unroll
        for (int u = 0; u < TH; ++u)
#pragma unroll
          for (int c = 0; c < 8; ++c) sq[u][c] = *reinterpret_cast<const f32x4*>(p.ssq_in + (int64_t)tcl[t0 + u] * PSSQ + e0 + c * 4);
#pragma unroll
        for (int u = 0; u < TH; ++u)
#pragma unroll
          for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) ss[u] += (e0 + c * 4 + e < p.n_ssq_in) ? sq[u][c][e] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < TH; ++u) scale[t0 + u] = rsqrtf(ss[u] * p.inv_dim + p.eps) * p.wfactor;
    }
  }
  f32x4 gv[4][4];  // next norm's gain for this lane's 16 x 4 rows (residual epilogue); gains of the head normalisation (QKV)
  if constexpr (EPI == PEPI_QKV && QKN) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int rg = min(rg_w + rb * 2 + (q4 >> 1), p.NRG - 1);
        const int n0 = rg * 16 + (q4 & 1) * 8 + hsel * 4;
        gv[rb][q4] = *reinterpret_cast<const f32x4*>(p.qk_gain + (n0 / p.hd < p.Hq ? 0 : p.hd) + n0 % p.hd);  // (value rows: unused)
      }
  }
  if constexpr (EPI == PEPI_RESID) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int rg = min(rg_w + rb * 2 + (q4 >> 1), p.NRG - 1);
        gv[rb][q4] = *reinterpret_cast<const f32x4*>(p.gain_next + rg * 16 + (q4 & 1) * 8 + hsel * 4);
      }
  }
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    __builtin_amdgcn_sched_barrier(0);  // one token group at a time: keeps the accumulator copies of the others out of the way
    const int t = tcl[tb];
    const bool ok = tok_ok[tb];
    const int64_t slot = kv_slot_in_block(blk[tb], pos[tb]);
    const int64_t kvbase = (slot / KV_BS) * p.Hkv;
    const int tok = (int)(slot % KV_BS);
    // one batch of loads for this token group: residual rows (RESID) or rotary factors (QKV)
    f32x4 pre[4][4];
    if constexpr (EPI != PEPI_SWIGLU) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int rg = min(rg_w + rb * 2 + (q4 >> 1), p.NRG - 1);
          const int n0 = rg * 16 + (q4 & 1) * 8 + hsel * 4;
          if constexpr (EPI == PEPI_RESID)  // (whole tiles are allocated: in bounds also for tokens and rows past the end)
            pre[rb][q4] = *reinterpret_cast<const f32x4*>(p.hp + image(tb, rb, q4));
          else pre[rb][q4] = *reinterpret_cast<const f32x4*>(p.rope + (int64_t)pos[tb] * (p.hd / 2) + ((n0 % p.hd) >> 1));
        }
    }
    float ssq_tok = 0.f;
    // Normalised query / key heads: a wavefront's 128 rows are one head of 128 or two heads of 64 (row blocks 0,1 and
    // 2,3), and a token's values of these rows sit in the two lanes l, l + 32: 1 / rms per head from the lane's own
    // squares and one cross-lane exchange.
    float head_rs[2] = {1.f, 1.f};
    if constexpr (EPI == PEPI_QKV && QKN) {
      float ss[2] = {0.f, 0.f};
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float v = acc[rb][tb][i] * scale[tb];
          ss[rb >> 1] += v * v;
        }
      if (p.hd == 128) ss[0] = ss[1] = ss[0] + ss[1];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        ss[hh] += __shfl_xor(ss[hh], 32);
        head_rs[hh] = rsqrtf(ss[hh] / (float)p.hd + p.eps);
      }
    }
    // QKV: finish the values in place (RMSNorm factor, head normalisation, rotation) and take the largest magnitude of
    // each head's vector for this token: the scale of its key / value codes.  A wavefront's 128 rows are one head of
    // 128 or two of 64 (row blocks 0,1 and 2,3); the token's values sit in the lanes l and l + 32.
    float head_amax[2] = {0.f, 0.f};
    if constexpr (EPI == PEPI_QKV) {
      const int rot_rows = (p.Hq + p.Hkv) * p.hd;
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int rg = rg_w + rb * 2 + (q4 >> 1);
          const int n0 = rg * 16 + (q4 & 1) * 8 + hsel * 4;
          float v4[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v4[i] = acc[rb][tb][q4 * 4 + i] * scale[tb];
          if (n0 < rot_rows) {
            if constexpr (QKN) {
#pragma unroll
              for (int i = 0; i < 4; ++i) v4[i] *= head_rs[rb >> 1] * gv[rb][q4][i];
            }
            const f32x4 cs = pre[rb][q4];  // (cos, sin) of the two rotary pairs held here
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
              float a = v4[2 * pr], b = v4[2 * pr + 1];
              v4[2 * pr] = a * cs[2 * pr] - b * cs[2 * pr + 1];
              v4[2 * pr + 1] = b * cs[2 * pr] + a * cs[2 * pr + 1];
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[rb][tb][q4 * 4 + i] = v4[i];
            head_amax[rb >> 1] = fmaxf(head_amax[rb >> 1], __builtin_fabsf(v4[i]));
          }
        }
      if (p.hd == 128) head_amax[0] = head_amax[1] = fmaxf(head_amax[0], head_amax[1]);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) head_amax[hh] = fmaxf(head_amax[hh], __shfl_xor(head_amax[hh], 32));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const int rgb = rg_w + rb * 2;  // first of the two row groups of this 32-row block
      if constexpr (EPI == PEPI_SWIGLU) {
        if (!ok || rgb + 1 >= p.NRG) continue;
#pragma unroll
        for (int q4 = 0; q4 < 2; ++q4) {
          int f0 = (rgb >> 1) * 16 + q4 * 8 + hsel * 4;
          union { uint16_t s[4]; u32x2 v; } o;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float g = acc[rb][tb][q4 * 4 + i] * scale[tb], u = acc[rb][tb][(q4 + 2) * 4 + i] * scale[tb];
            // (hardware reciprocal, 1 ulp: the result is rounded to fp16 right away; a correctly rounded fp32 division
            // costs ten instructions per element of the widest GEMM's epilogue)
            o.s[i] = f32_to_f16_sat(g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * u);
          }
          *reinterpret_cast<u32x2*>(p.ap + packed_p_offset(t, f0, p.Fp >> 4)) = o.v;
        }
      } else {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int rg = rgb + (q4 >> 1);
          if (!ok || rg >= p.NRG) continue;
          const int n0 = rg * 16 + (q4 & 1) * 8 + hsel * 4;
          float v4[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v4[i] = acc[rb][tb][q4 * 4 + i] * scale[tb];
          if constexpr (EPI == PEPI_RESID) {
            const f32x4 hv = pre[rb][q4], g4 = gv[rb][q4];
            const float hn[4] = {hv[0] + v4[0], hv[1] + v4[1], hv[2] + v4[2], hv[3] + v4[3]};
            *reinterpret_cast<float4*>(p.hp + image(tb, rb, q4)) = make_float4(hn[0], hn[1], hn[2], hn[3]);
            union { uint16_t s[4]; u32x2 v; } o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              ssq_tok += hn[i] * hn[i];
              o.s[i] = f32_to_f16_sat(hn[i] * g4[i]);
            }
            *reinterpret_cast<u32x2*>(p.xn_out + packed_p_offset(t, n0, p.d >> 4)) = o.v;
          } else {  // PEPI_QKV: the values were finished in place above
            const int head = n0 / p.hd, c0 = n0 % p.hd;
#pragma unroll
            for (int i = 0; i < 4; ++i) v4[i] = acc[rb][tb][q4 * 4 + i];
            union { uint16_t s[4]; u32x2 v; } o;
            if (head < p.Hq) {
#pragma unroll
              for (int i = 0; i < 4; ++i) o.s[i] = f32_to_f16_sat(v4[i]);  // queries feed the fp16 attention kernel
              *reinterpret_cast<u32x2*>(p.qp + (int64_t)t * (p.Hq * p.hd) + n0) = o.v;
            } else if (!LAST || !keep_cache[tb]) {
              // keys and values go to the cache as 16-bit codes with the scale of their (token, head) vector
              const bool is_v = head >= p.Hq + p.Hkv;
              const int j = head - p.Hq - (is_v ? p.Hkv : 0);
              const float amax = head_amax[rb >> 1], inv = kv_code_inv(amax);
#pragma unroll
              for (int i = 0; i < 4; ++i) o.s[i] = kv_code(v4[i], inv);
              if (!is_v) {
                *reinterpret_cast<u32x2*>(p.kplane + (kvbase + j) * (int64_t)(KV_BS * p.hd) + k_cache_offset(tok, c0)) = o.v;
              } else {
                uint16_t* dst = p.vplane + (kvbase + j) * (int64_t)(KV_BS * p.hd);
#pragma unroll
                for (int i = 0; i < 4; ++i) dst[v_cache_offset(tok, c0 + i)] = o.s[i];
              }
              if (c0 == 0) p.kvscale[kv_scale_offset(slot / KV_BS, p.Hkv, j) + (is_v ? 16 : 0) + tok] = kv_code_scale(amax);
            }
          }
        }
      }
    }
    if constexpr (EPI == PEPI_RESID) {
      ssq_tok += __shfl_xor(ssq_tok, 32);  // the two lane halves hold different rows of the same token
      sum_out(tb, ssq_tok);
    }
  }
}

// Epilogue of the token groups of last positions.  Before the epilogue above, a wavefront adds the hi and lo products of its
// groups and parks the sums in LDS, [group][4 rows][sequence] in units of 16 bytes (park_last); behind it, when the accumulators
// are free, it takes one group after the other from there (lane = sequence lane % 16 and row quads 4 q + lane / 16) and writes
// what the decode path's GEMMs write.  (In one with the epilogue above the 256 x 256 tiles spill up to 290 registers.)
#define LAST_UNITS 512  // of one group
template <int TB>
__device__ __forceinline__ void park_last(const PGemmP& p, f32x16 (&acc)[4][TB], int t_w, f32x4* lds) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    if (t_w + tb * 32 < p.first_last) continue;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[rb][tb][q4 * 4 + e] + __shfl_xor(acc[rb][tb][q4 * 4 + e], 16);
        if (!(lane & 16)) lds[tb * LAST_UNITS + (rb * 8 + q4 * 2 + (lane >> 5)) * 16 + (lane & 15)] = v;
      }
  }
}
// sum_out(tb, column, s): sum of squares of a sequence's new residual over the wavefront's rows, for both of its columns.
template <int EPI, bool QKN, int TB, typename SUM>
__device__ __forceinline__ void last_epilogue(const PGemmP& p, int rg_w, int t_w, const f32x4* lds, SUM sum_out) {
  const int lane = threadIdx.x & 63, s16 = lane & 15, part = lane >> 4;
#pragma unroll 1
  for (int tb = 0; tb < TB; ++tb, lds += LAST_UNITS) {
    const int at = t_w + tb * 32 - p.first_last;
    if (at < 0 || (at >> 1) >= p.n_last) continue;
    const int seq = (at >> 1) + s16;
    const bool ok = seq < p.n_last;
    const int sc = min(seq, p.n_last - 1), row = last_row_of(p.first_last, sc);
    float scale = p.wfactor;
    if (EPI != PEPI_RESID && p.ssq_in) {
      float ss = 0.f;
      for (int e0 = 0; e0 < p.n_ssq_in; e0 += 32) {
        f32x4 sq[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) sq[c] = *reinterpret_cast<const f32x4*>(p.ssq_in + (int64_t)row * PSSQ + e0 + c * 4);
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) ss += e0 + c * 4 + e < p.n_ssq_in ? sq[c][e] : 0.f;
      }
      scale *= rsqrtf(ss * p.inv_dim + p.eps);
    }
    auto value = [&](int quad) __attribute__((always_inline)) { return lds[quad * 16 + s16] * scale; };
    auto split4 = [&](f32x4 v, u32x2& hi, u32x2& lo) __attribute__((always_inline)) {
      union { uint16_t s[4]; u32x2 v; } h, l;
#pragma unroll
      for (int e = 0; e < 4; ++e) split_f16(v[e], h.s[e], l.s[e]);
      hi = h.v;
      lo = l.v;
    };
    u32x2 hi, lo;
    if constexpr (EPI == PEPI_SWIGLU) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const f32x4 g = value(rb * 8 + part), u = value(rb * 8 + 4 + part);
        f32x4 a;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = g[e] / (1.f + __expf(-g[e])) * u[e];
        split4(a, hi, lo);
        if (!ok || rg_w + rb * 2 + 1 >= p.NRG) continue;
        const int f0 = ((rg_w >> 1) + rb) * 16 + part * 4;
        *reinterpret_cast<u32x2*>(p.ap + packed_p_offset(row, f0, p.Fp >> 4)) = hi;
        *reinterpret_cast<u32x2*>(p.ap + packed_p_offset(row + 16, f0, p.Fp >> 4)) = lo;
      }
    } else if constexpr (EPI == PEPI_RESID) {
      float ss = 0.f;
      f32x4 hv[8], gv[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int n0 = min(rg_w + q, p.NRG - 1) * 16 + part * 4;
        hv[q] = *reinterpret_cast<const f32x4*>(p.h_last + (int64_t)sc * p.d + n0);
        gv[q] = *reinterpret_cast<const f32x4*>(p.gain_next + n0);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {  // row group rg_w + q
        if (rg_w + q >= p.NRG) break;
        const int n0 = (rg_w + q) * 16 + part * 4;
        const f32x4 hn = hv[q] + value(q * 4 + part);
        ss += hn[0] * hn[0] + hn[1] * hn[1] + hn[2] * hn[2] + hn[3] * hn[3];
        split4(hn * gv[q], hi, lo);
        if (!ok) continue;
        *reinterpret_cast<f32x4*>(p.h_last + (int64_t)sc * p.d + n0) = hn;
        *reinterpret_cast<u32x2*>(p.xn_out + packed_p_offset(row, n0, p.d >> 4)) = hi;
        *reinterpret_cast<u32x2*>(p.xn_out + packed_p_offset(row + 16, n0, p.d >> 4)) = lo;
      }
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (lane < 32) sum_out(tb, lane, ss);
    } else {
      const int pos = p.row_pos[row];
      const int64_t slot = kv_slot(p.table + (int64_t)sc * p.mbs, pos), blk = slot / KV_BS;
      const int tok = (int)(slot % KV_BS);
      f32x4 v[8];
      float ss[2] = {0.f, 0.f}, amax[2] = {0.f, 0.f};  // a head of 128, or two of 64
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        v[q] = value(q * 4 + part);
        if constexpr (QKN) ss[q >> 2] += v[q][0] * v[q][0] + v[q][1] * v[q][1] + v[q][2] * v[q][2] + v[q][3] * v[q][3];
      }
      if constexpr (QKN) {
        if (p.hd == 128) ss[0] = ss[1] = ss[0] + ss[1];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          ss[hh] += __shfl_xor(ss[hh], 16);
          ss[hh] += __shfl_xor(ss[hh], 32);
          ss[hh] = rsqrtf(ss[hh] / (float)p.hd + p.eps);
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int n0 = min(rg_w + q, p.NRG - 1) * 16 + part * 4;
        if (n0 < (p.Hq + p.Hkv) * p.hd) {
          if constexpr (QKN) v[q] *= *reinterpret_cast<const f32x4*>(p.qk_gain + (n0 / p.hd < p.Hq ? 0 : p.hd) + n0 % p.hd) * ss[q >> 2];
          const f32x4 cs = *reinterpret_cast<const f32x4*>(p.rope + (int64_t)pos * (p.hd / 2) + ((n0 % p.hd) >> 1));
#pragma unroll
          for (int pr = 0; pr < 2; ++pr) {
            const float a = v[q][2 * pr], b = v[q][2 * pr + 1];
            v[q][2 * pr] = a * cs[2 * pr] - b * cs[2 * pr + 1];
            v[q][2 * pr + 1] = b * cs[2 * pr] + a * cs[2 * pr + 1];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) amax[q >> 2] = fmaxf(amax[q >> 2], __builtin_fabsf(v[q][e]));
      }
      if (p.hd == 128) amax[0] = amax[1] = fmaxf(amax[0], amax[1]);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        amax[hh] = fmaxf(amax[hh], __shfl_xor(amax[hh], 16));
        amax[hh] = fmaxf(amax[hh], __shfl_xor(amax[hh], 32));
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (!ok || rg_w + q >= p.NRG) continue;
        const int n0 = (rg_w + q) * 16 + part * 4, head = n0 / p.hd, c0 = n0 % p.hd;
        if (head < p.Hq) {  // pre-scaled, for the decode attention
          split4(v[q] * p.qscale, hi, lo);
          *reinterpret_cast<u32x2*>(p.q_hi + (int64_t)sc * (p.Hq * p.hd) + n0) = hi;
          *reinterpret_cast<u32x2*>(p.q_lo + (int64_t)sc * (p.Hq * p.hd) + n0) = lo;
          continue;
        }
        const bool is_v = head >= p.Hq + p.Hkv;
        const int j = head - p.Hq - (is_v ? p.Hkv : 0);
        const float am = amax[q >> 2], inv = kv_code_inv(am);
        union { uint16_t s[4]; u32x2 v; } o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o.s[e] = kv_code(v[q][e], inv);
        uint16_t* dst = (is_v ? p.vplane : p.kplane) + (blk * p.Hkv + j) * (int64_t)(KV_BS * p.hd);
        if (!is_v) {
          *reinterpret_cast<u32x2*>(dst + k_cache_offset(tok, c0)) = o.v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[v_cache_offset(tok, c0 + e)] = o.s[e];
        }
        if (c0 == 0) p.kvscale[kv_scale_offset(blk, p.Hkv, j) + (is_v ? 16 : 0) + tok] = kv_code_scale(am);
      }
    }
  }
}

// QKN: the QKV epilogue also normalises the query and key heads (an instantiation of its own, so that the plain model's
// kernel carries none of its registers)
// TB: groups of 32 tokens per wavefront, 4 (256 tokens per tile) or 3 (192).  A k block of 32 columns takes 0.73 - 0.76 us with 256
// tokens and 0.53 (one round of workgroups) to 0.60 with 192, in either case about what the matrix cores need at the clock the
// power limit leaves them; the narrower tile serves calls whose tokens or rounds of workgroups it fits better (choose_pgemm): 8B
// shape, gate/up of 333 tokens 93 -> 78 us, whole prompts of 333, 700, 1100 and 3000 tokens 8525 -> 8240, 14 222 -> 13 590, 19 645
// -> 19 100 and 44 880 -> 42 120; 2000 tokens, five rounds against four of 256, 27 230 -> 27 340, so those keep the wide tile.
template <int EPI, bool QKN, bool LAST, int TB>
__global__ __launch_bounds__(256) void prefill_gemm_kernel(const PGemmP p) {
  // PGEMM_NB stage buffers of SB sixteen-byte units: 0..1023 weights [16 row groups][64], from 1024 on activations [2 TB token groups][2 k16][64]
  constexpr int SB = 1024 + 256 * TB, U = 4 + TB;  // U: units of 64 that each wavefront copies per block
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wn = wave >> 1, wt = wave & 1;

  int tt, rt;
  pgemm_tile_of((int)blockIdx.x, p.n_tt, p.n_rt, &tt, &rt);

  const int rg_tile = rt * 16;
  const int K16 = p.KB * 2;

  f32x16 acc[4][TB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  // Stage copies go from memory straight into LDS, without a register stage and without LDS store instructions: one
  // global_load_lds_dwordx4 moves 64 lanes x 16 bytes to 1 KiB of LDS in lane order (M0 = LDS byte address), which is
  // the layout of a packed fragment unit.  The copies are written as inline assembly so that the waits for them can be
  // placed by hand: the compiler would wait for all of them at every LDS barrier.  They count in vmcnt like any load
  // and complete in order; the kernel issues no other vector memory instruction before the end of the main loop.
  // NB stage buffers: while k block s is multiplied, blocks s+1 .. s+NB-2 are in flight or have landed and block
  // s+NB-1 is being requested.
  constexpr int NB = PGEMM_NB;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const u32x4* srcA[4];
  const u32x4* srcB[TB];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = wave_u + 4 * i;  // fragment unit handled by this wavefront: 0..15, activations 0 .. 4 TB - 1
    srcA[i] = p.W + (int64_t)min(rg_tile + f, p.NRG - 1) * 64;
    if (i < TB) srcB[i] = p.X + ((int64_t)(tt * (2 * TB) + (f >> 1)) * K16 + (f & 1)) * 64;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t voff = lane * 16;
  u32x4 fa0[4], fb0[TB], fa1[4], fb1[TB];
  const int fm = lane & 31, fh = lane >> 5;
  auto dma16 = [&](const u32x4* g, uint32_t lds_addr) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(g), "s"(lds_addr) : "memory", "m0");
  };
  // unit i = 0 .. U - 1 of this wavefront's share of a k block: even = weights, odd = activations
  auto stage1 = [&](int kbc, int buf, int i) __attribute__((always_inline)) {
    const int q = i >> 1;
    if (i & 1) dma16(srcB[q] + (int64_t)kbc * 128, lds0 + (uint32_t)(buf * SB + 1024 + (wave_u + 4 * q) * 64) * 16u);
    else dma16(srcA[q] + (int64_t)kbc * p.NRG * 64, lds0 + (uint32_t)(buf * SB + (wave_u + 4 * q) * 64) * 16u);
  };
  auto stage = [&](int kb, int buf) __attribute__((always_inline)) {
    const int kbc = min(kb, p.KB - 1);
#pragma unroll
    for (int i = 0; i < U; ++i) stage1(kbc, buf, i);
  };
  // fragment read i = 0 .. U - 1 of a 16-column half: 0..3 weights (row blocks), then activations (token blocks)
  auto fetch1 = [&](u32x4(&fa)[4], u32x4(&fb)[TB], int buf, int k16, int i) __attribute__((always_inline)) {
    if (i < 4) fa[i] = smem[buf * SB + (wn * 8 + i * 2 + (fm >> 4)) * 64 + ((k16 * 2 + fh) << 4) + (fm & 15)];
    else fb[i - 4] = smem[buf * SB + 1024 + ((wt * TB + (i - 4)) * 2 + k16) * 64 + lane];
  };
  auto fetch = [&](u32x4(&fa)[4], u32x4(&fb)[TB], int buf, int k16) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < U; ++i) fetch1(fa, fb, buf, k16, i);
  };
  auto mfma1 = [&](u32x4(&fa)[4], u32x4(&fb)[TB], int i) __attribute__((always_inline)) {
    const int rb = i / TB, tb = i % TB;
    acc[rb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(fa[rb]), as_f16x8(fb[tb]), acc[rb][tb], 0, 0, 0);
  };
  auto lds_barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  // k block s sits in buffer r = s mod NB; two fragment sets carry the LDS reads of its two 16-column halves.  The
  // instruction order is fixed by hand: one LDS read behind each of the first U MFMAs of a half (half 1 of block s
  // in the first half, half 0 of block s+1 in the second, each 8 to 16 MFMAs before its data is needed) and one stage
  // copy behind every fourth MFMA (TB in the first half of a block, four in the second), so that the requests of the four wavefronts reach the memory pipeline evenly spread.
  // The copies of block s+NB-1 go to the buffer of block s-1, which nobody reads any more once the barrier of block
  // s-1 has been passed.  One barrier per k block, in the middle: in front of it a wavefront waits until its own units
  // of block s+1 have landed (at most (NB-3) blocks of U units and the TB units of block s+NB-1 requested so far may
  // still be outstanding); behind it everybody's have.  Past the last k block the copies are redirected to the last
  // block; nobody reads them.
  // s_waitcnt immediates for "at most n memory requests outstanding": a 6-bit count split over bits 3:0 and 15:14, the
  // other counters unconstrained
  constexpr int VM_MID = (NB - 3) * U + TB;
  constexpr int WAIT_MID = 0x0F70 | (VM_MID & 15) | ((VM_MID >> 4) << 14);
  constexpr int VM_PRO = (NB - 2) * U;
  constexpr int WAIT_PRO = 0x0F70 | (VM_PRO & 15) | ((VM_PRO >> 4) << 14);
  auto k_block = [&](int s, int r) __attribute__((always_inline)) {
    const int buf1 = r == NB - 1 ? 0 : r + 1, bufp = r == 0 ? NB - 1 : r - 1;
    const int kbc = min(s + NB - 1, p.KB - 1);
#pragma unroll
    for (int i = 0; i < 4 * TB; ++i) {
      mfma1(fa0, fb0, i);
      if (i < U) fetch1(fa1, fb1, r, 1, i);
      if ((i & 3) == 3) stage1(kbc, bufp, i >> 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(WAIT_MID);  // this wavefront's units of block s+1 have landed
    lds_barrier();                         // ... everybody's
#pragma unroll
    for (int i = 0; i < 4 * TB; ++i) {
      mfma1(fa1, fb1, i);
      if (i < U) fetch1(fa0, fb0, buf1, 0, i);
      if (i % TB == TB - 1) stage1(kbc, bufp, TB + i / TB);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int b = 0; b < NB - 1; ++b) stage(b, b);
  __builtin_amdgcn_s_waitcnt(WAIT_PRO);
  lds_barrier();
  fetch(fa0, fb0, 0, 0);
  {
    int s = 0;
    for (; s + NB - 1 < p.KB; s += NB) {
#pragma unroll
      for (int r = 0; r < NB; ++r) k_block(s + r, r);
    }
#pragma unroll
    for (int r = 0; r < NB - 1; ++r)
      if (s + r < p.KB) k_block(s + r, r);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the redirected copies past the last k block have landed too
  __syncthreads();  // the staging buffers are dead from here on; the residual epilogue reuses them
  float(*red_ssq)[256] = reinterpret_cast<float(*)[256]>(smem);
  (void)red_ssq;

  const int t_w = __builtin_amdgcn_readfirstlane((tt * 2 + wt) * 32 * TB), g32 = (tt * 2 + wt) * TB;  // first token, group of 32
  f32x4* parked = reinterpret_cast<f32x4*>(smem + 128 + wave * TB * LAST_UNITS);
  if constexpr (LAST) park_last(p, acc, t_w, parked);
  if (!LAST || t_w < p.first_last) pgemm_epilogue<EPI, QKN, TB, LAST>(p, acc, g32 >> 3, rt, wn, (g32 >> 2) & 1, g32 & 3, [&](int tb, float ssq_tok) __attribute__((always_inline)) {
    const int at = (wt * TB + tb) * 32 + lane;
    if (lane < 32 && (!LAST || tt * 64 * TB + at < p.first_last)) red_ssq[wn][at] = ssq_tok;  // (slots of tokens past the end are never read)
  });
  if constexpr (LAST) {
    __syncthreads();
    last_epilogue<EPI, QKN, TB>(p, rt * 16 + wn * 8, t_w, parked, [&](int tb, int c, float s) __attribute__((always_inline)) { red_ssq[wn][(wt * TB + tb) * 32 + c] = s; });
  }
  if constexpr (EPI == PEPI_RESID) {
    // per (row tile, token) sum of squares of the new residual, the two row halves added in a fixed order
    __syncthreads();
    const int t = tt * 64 * TB + tid;
    if (tid < 64 * TB && t < p.T) p.ssq_out[(int64_t)t * PSSQ + rt] = red_ssq[0][tid] + red_ssq[1][tid];
  }
}

// ------------------------------------------------------------------------------------------------
// The same GEMM with tiles of 128 rows x 128 TB tokens: four wavefronts of 128 rows x 32 TB tokens, and the k range of a
// tile cut over ksplit workgroups where the tiles alone leave compute units idle.
// The four wavefronts share the weight fragments (through LDS, copied as above) but no activations: those go from memory
// straight into the registers of the one wavefront that needs them, PSG_D / TB blocks of 64 columns ahead.
// Bound by what one compute unit takes in, 50 - 55 KB per us: a k block of 32 columns takes 0.29 us (TB = 1, 16 KB) or 0.43
// us (TB = 2, 24 KB) with few or many workgroups, with the activations through LDS as well, and with two or five blocks in
// flight; the 256 x 256 tiles (32 KB) take 0.7 - 0.76 us.  Up to 128 tokens the weights are read once: 4096 x 14336 weights,
// 128 tokens, 8 splits: 37 us against 256 with 16 workgroups of 256 x 256 tiles.  (The wavefront's waits: 48 % of its
// cycles at 512 tokens, matrix cores busy 49 %, bank conflicts none.)
// All splits of a tile get workgroup ids that are equal modulo 8 and hand their partial tiles over like the decode GEMMs
// (device-scope accesses, explicit wait, counter; the last one adds them in split order).  Token tiles are innermost, in
// groups of 8: they run side by side behind one L2 and share the weights.
#define PSG_NB 8  // stage buffers of 64 columns of the tile's weights (16 KiB each)
#define PSG_D 8
#define PSG_LDS_BYTES (PSG_NB * 1024 * 16)
template <int EPI, bool QKN, int TB, bool LAST>
__global__ __launch_bounds__(256, 1) void prefill_gemm_small_kernel(const PGemmP p) {
  extern __shared__ u32x4 smem[];  // per stage 1024 units: [2 k blocks][8 row groups][64]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int slot = blockIdx.x >> 3;
  const int per_group = (p.n_rt128 + 7) / 8 * p.ksplit * 8;
  const int group = slot / per_group, in_group = slot - group * per_group;
  const int gsz = min(8, p.n_ttS - group * 8);  // (only the last group is narrower)
  const int tt1 = group * 8 + in_group % gsz, split = (in_group / gsz) % p.ksplit;
  const int rt1 = (blockIdx.x & 7) + 8 * (in_group / (gsz * p.ksplit));
  if (rt1 >= p.n_rt128) return;  // grid padding when the row tiles are not a multiple of 8
  const int rg_tile = rt1 * 8, K16 = p.KB * 2;
  const int kb_begin = split * p.kb_per_split, nkb = min(p.KB, kb_begin + p.kb_per_split) - kb_begin;
  // token groups of this wavefront that hold tokens of the call; one without any only helps with the copies
  const int t_w = tt1 * 128 * TB + __builtin_amdgcn_readfirstlane(wave) * 32 * TB;
  const int n_act = min(TB, max(0, (p.T - t_w + 31) >> 5));

  f32x16 acc[4][TB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  // Stage copies, buffers and waits as in prefill_gemm_kernel, in blocks of 64 columns (four steps of 16); a wavefront
  // moves 4 of a block's 16 units, one per step.  The activations are ordinary loads, whose waits the compiler places; they
  // count in vmcnt too, so the hand-placed waits, which allow for the copies alone, wait for somewhat more than they need.
  constexpr int NB = PSG_NB, D = PSG_D / TB;
  static_assert(NB % D == 0, "the register sets rotate with the unrolled loop");
  const int nsb = (nkb + 1) >> 1;  // blocks; the last one may be half empty
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const u32x4* srcA[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) srcA[i] = p.W + ((int64_t)kb_begin * p.NRG + min(rg_tile + wave_u + 4 * i, p.NRG - 1)) * 64;
  const u32x4* srcB[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) srcB[tb] = p.X + ((int64_t)((tt1 * 4 + wave_u) * TB + tb) * K16 + (int64_t)kb_begin * 2) * 64;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t voff = lane * 16;
  u32x4 fa[2][4], fb[D][4][TB];
  const int fm = lane & 31, fh = lane >> 5;
  auto stage1 = [&](int sb, int buf, int i) __attribute__((always_inline)) {
    const u32x4* g = srcA[i & 1] + (int64_t)min(sb * 2 + (i >> 1), nkb - 1) * p.NRG * 64;
    const uint32_t lds_addr = lds0 + (uint32_t)(buf * 1024 + (i >> 1) * 512 + (wave_u + 4 * (i & 1)) * 64) * 16u;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(g), "s"(lds_addr) : "memory", "m0");
  };
  auto load_b = [&](u32x4(&f)[TB], int sb, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) f[tb] = srcB[tb][(int64_t)min(sb * 4 + t, nkb * 2 - 1) * 64 + lane];
  };
  auto fetch1 = [&](u32x4(&f)[4], int buf, int t, int rb) __attribute__((always_inline)) {
    f[rb] = smem[buf * 1024 + (t >> 1) * 512 + (rb * 2 + (fm >> 4)) * 64 + (((t & 1) * 2 + fh) << 4) + (fm & 15)];
  };
  auto lds_barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  // requests that may still be outstanding when block s+1 (the first block) has to have landed
  constexpr int VM_MID = (NB - 3) * 4 + 3, VM_PRO = (NB - 2) * 4;
  constexpr int WAIT_MID = 0x0F70 | (VM_MID & 15) | ((VM_MID >> 4) << 14);
  constexpr int WAIT_PRO = 0x0F70 | (VM_PRO & 15) | ((VM_PRO >> 4) << 14);
  auto loop = [&](auto act) __attribute__((always_inline)) {
    constexpr bool ACT = decltype(act)::value;  // this wavefront has tokens
    // block s in buffer r, activations in register set r % D.  Per step: the MFMAs of its 16 columns, the weight fragments
    // of the next step behind the first four, then the activations of block s + D into the registers just used, and
    // one stage copy of block s + NB - 1 into the buffer of block s - 1.
    auto block = [&](int s, int r, auto tail) __attribute__((always_inline)) {
      const int buf1 = r == NB - 1 ? 0 : r + 1, bufp = r == 0 ? NB - 1 : r - 1;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t == 3) {
          __builtin_amdgcn_s_waitcnt(WAIT_MID);  // this wavefront's units of block s+1 have landed
          lds_barrier();                         // ... everybody's
        }
        if (ACT) {
          const bool skip = decltype(tail)::value && t >= 2 && s * 2 + 2 > nkb;  // the empty half of the last block
#pragma unroll
          for (int i = 0; i < 4 * TB; ++i) {
            const int rb = i & 3, tb = i >> 2;
            if (!skip) acc[rb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(fa[t & 1][rb]), as_f16x8(fb[r % D][t][tb]), acc[rb][tb], 0, 0, 0);
            if (i < 4) fetch1(fa[(t + 1) & 1], t == 3 ? buf1 : r, (t + 1) & 3, i);
            __builtin_amdgcn_sched_barrier(0);
          }
          load_b(fb[r % D][t], s + D, t);
        }
        stage1(s + NB - 1, bufp, t);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (ACT) {
#pragma unroll
      for (int s = 0; s < D; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) load_b(fb[s][t], s, t);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB - 1; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) stage1(b, b, i);
    __builtin_amdgcn_s_waitcnt(WAIT_PRO);
    lds_barrier();
    if (ACT) {
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) fetch1(fa[0], 0, 0, rb);
    }
    int s = 0;
    for (; s + NB < nsb; s += NB) {
#pragma unroll
      for (int r = 0; r < NB; ++r) block(s + r, r, std::false_type{});
    }
#pragma unroll
    for (int r = 0; r < NB; ++r)
      if (s + r < nsb) block(s + r, r, std::true_type{});
  };
  if (n_act) loop(std::true_type{});
  else loop(std::false_type{});
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the redirected copies past the last k block have landed too
  __syncthreads();                     // the staging buffers are dead from here on

  if (p.ksplit > 1) {
    volatile int* s_last = reinterpret_cast<volatile int*>(smem);
    const __amdgpu_buffer_rsrc_t prs = shared_rsrc(p.partial);
    const int tile = tt1 * p.n_rt128 + rt1;
    // register image: [split][tile][wavefront][token group][16 units][lane] of 16 bytes
    auto punit = [&](int sp, int tb, int u) __attribute__((always_inline)) {
      return (uint32_t)(((((sp * (p.n_ttS * p.n_rt128) + tile) * 4 + wave) * TB + tb) * 16 + u) * 64 + lane) * 16u;
    };
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      if (tb >= n_act) break;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int i = (u & 3) * 4;
        const f32x4 v = {acc[u >> 2][tb][i], acc[u >> 2][tb][i + 1], acc[u >> 2][tb][i + 2], acc[u >> 2][tb][i + 3]};
        store_shared_f32x4(prs, punit(split, tb, u), v);
      }
    }
    wait_own_memory_ops();
    __syncthreads();
    if (tid == 0) *s_last = arrive_last(&p.counters[tile], p.ksplit, p.fence_handover, p.fault_flag);
    __syncthreads();
    if (!*s_last) return;
    if (p.fence_handover) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid == 0) __hip_atomic_store(&p.counters[tile], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Added in split order (reproducible), two on their way at a time: a tile is 16 loads a lane, and with three the kernels were slower
    // (8B shape, O projection of 333 tokens 30.6 us with two and 32.7 with three, 8192 columns, 256 tokens, QKV 71.3 and 74.7).
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      if (tb >= n_act) break;
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][tb][i] = 0.f;
      f32x4 pv[2][16];
      add_in_order<2>(p.ksplit,
          [&](int w, int sp) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 16; ++u) pv[w][u] = load_shared_f32x4(prs, punit(sp, tb, u));
          },
          [&](int w) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 16; ++u)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[u >> 2][tb][(u & 3) * 4 + e] += pv[w][u][e];
          });
    }
  }
  if (n_act == 0) return;
  const int g32 = tt1 * 4 * TB + wave * TB;  // the wavefront's first group of 32 tokens; 8 of them make a 256-token tile
  f32x4* parked = reinterpret_cast<f32x4*>(smem + 64 + wave * TB * LAST_UNITS);  // (its own: no barrier needed; behind s_last)
  if constexpr (LAST) park_last(p, acc, t_w, parked);
  if (!LAST || t_w < p.first_last) pgemm_epilogue<EPI, QKN, TB, LAST>(p, acc, g32 >> 3, rt1 >> 1, rt1 & 1, (g32 >> 2) & 1, g32 & 3, [&](int tb, float ssq_tok) __attribute__((always_inline)) {
    const int t = t_w + tb * 32 + lane;
    if (lane < 32 && t < (LAST ? p.T_new : p.T)) p.ssq_out[(int64_t)t * PSSQ + rt1] = ssq_tok;
  });
  if constexpr (LAST) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    last_epilogue<EPI, QKN, TB>(p, rg_tile, t_w, parked, [&](int tb, int c, float s) __attribute__((always_inline)) { p.ssq_out[(int64_t)(t_w + tb * 32 + c) * PSSQ + rt1] = s; });
  }
}

// ------------------------------------------------------------------------------------------------
// Causal paged flash attention for new tokens.  One workgroup = 64 consecutive new tokens of one
// sequence x one kv head (x GH of its query heads); each wavefront owns 16 query positions and keeps
// S^T = K Q^T / O^T = V^T P^T for its GH heads.  The keys and values of a pair of blocks (32 keys) are
// copied into LDS once per workgroup and read from there by the four wavefronts (the cache already stores them
// in MFMA operand order; the copy turns the 16-bit codes into fp16 values, code * scale of its token, rounded once - the
// precision an fp16 cache would give this pass, which only needs the keys and values of other positions to matrix-core
// accuracy); the next pair travels from memory while this one is used.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Key range of a tile: a call with few tiles leaves compute units idle, so the key pairs of a tile are cut into up to
// max_splits ranges of at least PATTN_MIN_PAIRS pairs, each walked by a workgroup of its own that parks its softmax state;
// prefill_attn_merge_kernel then combines them.  A walk takes about 1.2 us per pair whatever the other compute units do: 16
// tokens over 6000 cached ones, 8 workgroups: 225 us per layer of the 8B shape, the call 26.4 ms; with 16 ranges (and the
// GEMMs of small calls) 8.4 ms.  At least 4, 8 or 16 pairs per range: 8.44, 8.60, 8.70 ms.
#define PATTN_MIN_PAIRS 4
#define PATTN_MAX_ITEMS 256  // calls with more workgroups than this are not cut
__host__ __device__ __forceinline__ int pattn_splits(int npairs, int max_splits) {
  const int n = npairs / PATTN_MIN_PAIRS;
  return n < 1 ? 1 : n < max_splits ? n : max_splits;
}
// floats a workgroup parks: [wavefront][query head][HD / 16][lane][4] unnormalised outputs, then [wavefront][query head][lane] (m, l)
constexpr int pattn_record(int HD, int GH, int HG) { return 4 * HG * GH * 64 * (HD / 4 + 2); }

template <int HD, int GH, int HG>
__global__ __launch_bounds__(256 * HG, 2 / HG) void prefill_attn_kernel(const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kplane,
                                                            const uint16_t* __restrict__ vplane, const float* __restrict__ kvscale,
                                                            const int32_t* __restrict__ q_lens,
                                                            const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ table,
                                                            int mbs, int Hq, int Hkv, int G, const int32_t* __restrict__ tile_seq,
                                                            const int32_t* __restrict__ tile_q0, const int32_t* __restrict__ meta,
                                                            const int32_t* __restrict__ cum_rows, float scale_log2,
                                                            uint16_t* __restrict__ op, int max_tiles, int max_splits,
                                                            float* __restrict__ part) {
  constexpr int NKF = HD / 32, NVF = HD / 16;
  constexpr int CH = NKF * 64;         // 16-byte units of one block's keys (and of one block's values)
  constexpr int NT = 256 * HG;         // threads: HG groups of four wavefronts, each group with its own GH query heads
  constexpr int NLD = 4 * CH / NT;     // units each thread moves per pair
  __shared__ u32x4 kv[2][4 * CH];      // per pair: keys of block 0, keys of block 1, values of block 0, values of block 1
  // Work items in the order (head group, kv head, key range, tile), tiles fastest; workgroup ids are dealt round-robin to the 8
  // XCDs, so the ids are transposed: XCD x gets the x-th eighth of that order, i.e. the consecutive tiles of a
  // sequence and kv head run behind one L2 and fetch its keys and values into it once (with 8 kv heads: one per XCD).
  int item = blockIdx.x;
  const int n_items = gridDim.x;
  if (n_items % 8 == 0) item = (item & 7) * (n_items >> 3) + (item >> 3);
  const int tile = item % max_tiles;
  if (tile >= meta[0]) return;
  const int split = (item / max_tiles) % max_splits, jh = item / (max_tiles * max_splits);  // (kv head, then head group)
  const int j = jh % Hkv;
  const int tid = threadIdx.x, wave = (tid >> 6) & 3, lane = tid & 63;
  const int h0 = j * G + ((jh / Hkv) * HG + (tid >> 8)) * GH;  // first query head handled by this wavefront
  const int n = lane & 15, g = lane >> 4;
  const int b = tile_seq[tile];
  const int qlen = q_lens[b], ctx = seq_lens[b];
  const int prefix = ctx - qlen;
  const int tq0 = tile_q0[tile];
  const int qw0 = tq0 + wave * 16;        // first query (index among the new tokens) of this wavefront
  const bool active = qw0 < qlen;         // a wavefront past the end of the sequence only helps with the copies
  const int nq = active ? min(16, qlen - qw0) : 1;
  const int64_t row0 = (int64_t)cum_rows[b] + (active ? qw0 : 0);
  const int my_q = min(n, nq - 1);        // lanes past the end repeat the last query; their output is dropped
  const int qpos = prefix + qw0 + my_q;   // this lane's query position
  const int kmax = active ? prefix + qw0 + nq : 0;  // keys 0 .. kmax-1 are visible to some query of the wavefront
  const int npairs = (kmax + 31) / 32;
  const int npairs_tile = (prefix + min(qlen, tq0 + 64) + 31) / 32;  // pairs of the tile ...
  const int nsplit = pattn_splits(npairs_tile, max_splits);
  if (split >= nsplit) return;
  const int per_split = (npairs_tile + nsplit - 1) / nsplit;
  const int pr_first = split * per_split;                            // ... and the ones this workgroup walks through
  const int npairs_wg = min(npairs_tile, pr_first + per_split);
  const int last_blk = (ctx - 1) / KV_BS;
  const int32_t* trow = table + (int64_t)b * mbs;
  const int QD = Hq * HD;

  f16x8 qf[GH][NKF];
#pragma unroll
  for (int hh = 0; hh < GH; ++hh)
#pragma unroll
    for (int f = 0; f < NKF; ++f)
      qf[hh][f] = as_f16x8(*reinterpret_cast<const u32x4*>(qp + (row0 + my_q) * QD + (h0 + hh) * HD + f * 32 + g * 8));

  f32x4 oacc[GH][NVF];
  float m_run[GH], l_run[GH];
#pragma unroll
  for (int hh = 0; hh < GH; ++hh) {
    m_run[hh] = NEG_INF;
    l_run[hh] = 0.f;
#pragma unroll
    for (int f = 0; f < NVF; ++f) oacc[hh][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int64_t blk_elems = (int64_t)KV_BS * HD;
  u32x4 stg[NLD];
  // units 0 .. NLD/2-1 of a thread are keys (one token per unit: one scale), the others values (four tokens per unit)
  static_assert(NLD % 2 == 0 && (NLD / 2) * NT == 2 * CH, "the first half of a thread's units are keys");
  float ksc[NLD / 2];
  f32x4 vsc[NLD / 2];
  // Block ids are fetched one pair ahead of the request that uses them, so the request never waits for the table.
  // A pair past the tile's last one is redirected to the last one (in bounds, never used).
  int id0 = 0, id1 = 0;
  auto fetch_ids = [&](int pr) __attribute__((always_inline)) {
    const int prc = min(pr, npairs_tile - 1);
    id0 = trow[min(prc * 2, last_blk)];
    id1 = trow[min(prc * 2 + 1, last_blk)];
  };
  auto request = [&]() __attribute__((always_inline)) {
    const int64_t off0 = ((int64_t)id0 * Hkv + j) * blk_elems;
    const int64_t off1 = ((int64_t)id1 * Hkv + j) * blk_elems;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int u = tid + i * NT, c = u / CH, within = u % CH;
      const uint16_t* src = (c < 2 ? kplane : vplane) + ((c & 1) ? off1 : off0) + within * 8;
      stg[i] = *reinterpret_cast<const u32x4*>(src);
      const float* sc = kvscale + kv_scale_offset((c & 1) ? id1 : id0, Hkv, j);
      if (i < NLD / 2) ksc[i] = sc[within & 15];                                        // key unit: token = unit % 16
      else vsc[i - NLD / 2] = *reinterpret_cast<const f32x4*>(sc + 16 + ((within >> 3) & 3) * 4);  // value unit: tokens 4t .. 4t+3
    }
  };
  auto copy_in = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const uint32_t w[4] = {stg[i].x, stg[i].y, stg[i].z, stg[i].w};
      u32x4 out;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        // word d holds elements 2d, 2d+1 of the unit; a value unit's element e belongs to token e % 4
        const float s0 = i < NLD / 2 ? ksc[i < NLD / 2 ? i : 0] : vsc[i < NLD / 2 ? 0 : i - NLD / 2][(2 * d) & 3];
        const float s1 = i < NLD / 2 ? ksc[i < NLD / 2 ? i : 0] : vsc[i < NLD / 2 ? 0 : i - NLD / 2][(2 * d + 1) & 3];
        // offset-binary codes u = q + 32768:  value = (u - 32768) * scale
        const float x0 = __builtin_fmaf((float)(w[d] & 0xffffu), s0, -32768.f * s0), x1 = __builtin_fmaf((float)(w[d] >> 16), s1, -32768.f * s1);
        const f16x2 h = __builtin_convertvector((f32x2){x0, x1}, f16x2);
        out[d] = __builtin_bit_cast(uint32_t, h);
      }
      kv[buf][tid + i * NT] = out;
    }
  };
  // masked = false: every key of the pair is visible to every query of the wavefront (the pair ends at or before its
  // first query position), so neither the scores nor the values need a mask; that is the case for all pairs but the
  // last one to three of a wavefront.  The argument is a literal at both call sites.
  auto compute = [&](int buf, int pr, const bool masked) __attribute__((always_inline)) {
    const int base = pr * 32;
    u32x4 kf0[NKF], kf1[NKF];
    u32x2 vf0[NVF], vf1[NVF];
    const u32x2* v0p = reinterpret_cast<const u32x2*>(&kv[buf][2 * CH]);
    const u32x2* v1p = reinterpret_cast<const u32x2*>(&kv[buf][3 * CH]);
#pragma unroll
    for (int f = 0; f < NKF; ++f) {
      kf0[f] = kv[buf][f * 64 + lane];
      kf1[f] = kv[buf][CH + f * 64 + lane];
    }
#pragma unroll
    for (int f = 0; f < NVF; ++f) {
      vf0[f] = v0p[f * 64 + lane];
      vf1[f] = v1p[f * 64 + lane];
    }
    // three passes over the GH heads (scores, softmax, values) rather than one head after the other: the heads are
    // independent, so each pass is a run of independent MFMAs or of independent cross-lane exchanges
    f32x4 s0[GH], s1[GH];
#pragma unroll
    for (int hh = 0; hh < GH; ++hh) {
      s0[hh] = f32x4{0.f, 0.f, 0.f, 0.f};
      s1[hh] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int f = 0; f < NKF; ++f)
#pragma unroll
      for (int hh = 0; hh < GH; ++hh) {
        s0[hh] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(kf0[f]), qf[hh][f], s0[hh], 0, 0, 0);
        s1[hh] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(kf1[f]), qf[hh][f], s1[hh], 0, 0, 0);
      }
    // Softmax numerators p = 2^(score * log2(e)/sqrt(hd) - m) with a per-query reference point m (m_run) that is not
    // necessarily the running maximum: the result o / l does not depend on it.  The common case takes no maximum at
    // all: the exponentials are formed against the current reference, and only if some lane's sum of its eight
    // numerators exceeds 256 (so a numerator might not fit fp16 comfortably; also true for a NaN or an infinity) or
    // while a query has no reference yet (on the first pair, or as long as it has seen hidden keys only) the wavefront takes the exact maxima, moves the reference up, rescales o
    // and l and forms the exponentials again.  After the first pairs of a sequence that is rare, and the 4 * NVF
    // accumulator registers per head are then left alone.  Hidden keys (later than the query, or slots past the end
    // of the sequence, which may hold anything) enter as -inf and get p = 0.
    f16x8 pbv[GH];
#pragma unroll
    for (int hh = 0; hh < GH; ++hh) {
      float sr[8];  // raw scores
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sr[i] = (!masked || base + 4 * g + i <= qpos) ? s0[hh][i] : NEG_INF;
        sr[4 + i] = (!masked || base + 16 + 4 * g + i <= qpos) ? s1[hh][i] : NEG_INF;
      }
      float neg_m = (m_run[hh] == NEG_INF) ? 0.f : -m_run[hh];
      float pv[8];
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pv[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sr[i], scale_log2, neg_m));
        psum += pv[i];
      }
      if (pr == pr_first || __any(!(psum <= 256.f) || (masked && m_run[hh] == NEG_INF))) {
        float scl[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) scl[i] = sr[i] * scale_log2;
        float mx = fmaxf(fmaxf(fmaxf(scl[0], scl[1]), fmaxf(scl[2], scl[3])), fmaxf(fmaxf(scl[4], scl[5]), fmaxf(scl[6], scl[7])));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run[hh], mx);
        // a query whose visible keys all lie in later pairs has m_new = -inf here: keep its state untouched
        const float alpha = __builtin_amdgcn_exp2f(m_run[hh] - ((m_new == NEG_INF) ? 0.f : m_new));
        l_run[hh] *= alpha;
        m_run[hh] = m_new;
#pragma unroll
        for (int f = 0; f < NVF; ++f) {
          oacc[hh][f][0] *= alpha; oacc[hh][f][1] *= alpha; oacc[hh][f][2] *= alpha; oacc[hh][f][3] *= alpha;
        }
        neg_m = (m_new == NEG_INF) ? 0.f : -m_new;
        psum = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(scl[i] + neg_m);
          psum += pv[i];
        }
      }
      l_run[hh] += psum;
      // two values per conversion instruction, round to nearest even
      const f16x2 h01 = __builtin_convertvector((f32x2){pv[0], pv[1]}, f16x2), h23 = __builtin_convertvector((f32x2){pv[2], pv[3]}, f16x2);
      const f16x2 h45 = __builtin_convertvector((f32x2){pv[4], pv[5]}, f16x2), h67 = __builtin_convertvector((f32x2){pv[6], pv[7]}, f16x2);
      pbv[hh] = __builtin_shufflevector(__builtin_shufflevector(h01, h23, 0, 1, 2, 3), __builtin_shufflevector(h45, h67, 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
    }
    // slots past the end of the sequence may hold anything: keep them out of the MFMA (masks are all-ones elsewhere)
    uint32_t a01 = 0xFFFFFFFFu, a23 = 0xFFFFFFFFu, b01 = 0xFFFFFFFFu, b23 = 0xFFFFFFFFu;
    if (masked) {
      const int ka = base + 4 * g, kb2 = base + 16 + 4 * g;
      a01 = (ka + 0 < ctx ? 0xFFFFu : 0u) | (ka + 1 < ctx ? 0xFFFF0000u : 0u);
      a23 = (ka + 2 < ctx ? 0xFFFFu : 0u) | (ka + 3 < ctx ? 0xFFFF0000u : 0u);
      b01 = (kb2 + 0 < ctx ? 0xFFFFu : 0u) | (kb2 + 1 < ctx ? 0xFFFF0000u : 0u);
      b23 = (kb2 + 2 < ctx ? 0xFFFFu : 0u) | (kb2 + 3 < ctx ? 0xFFFF0000u : 0u);
    }
#pragma unroll
    for (int f = 0; f < NVF; ++f) {
      const u32x4 a = masked ? u32x4{vf0[f].x & a01, vf0[f].y & a23, vf1[f].x & b01, vf1[f].y & b23}
                             : u32x4{vf0[f].x, vf0[f].y, vf1[f].x, vf1[f].y};
#pragma unroll
      for (int hh = 0; hh < GH; ++hh)
        oacc[hh][f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), pbv[hh], oacc[hh][f], 0, 0, 0);
    }
  };

  fetch_ids(pr_first);
  request();
  fetch_ids(pr_first + 1);
  copy_in(pr_first & 1);
  __syncthreads();
  for (int pr = pr_first; pr < npairs_wg; ++pr) {
    request();          // pair pr + 1
    fetch_ids(pr + 2);
    __builtin_amdgcn_sched_barrier(0);
    if (pr < npairs) {
      if (pr * 32 + 31 <= prefix + qw0) compute(pr & 1, pr, false);
      else compute(pr & 1, pr, true);
    }
    __builtin_amdgcn_sched_barrier(0);
    copy_in((pr + 1) & 1);
    __syncthreads();
  }
  if (nsplit > 1) {
    // a wavefront without visible keys in this range parks m = -inf, l = 0, o = 0
    float* rec = part + ((int64_t)(jh * max_tiles + tile) * max_splits + split) * pattn_record(HD, GH, HG);
    float* ml = rec + 4 * HG * GH * 64 * (HD / 4);
    const int w = tid >> 6;
#pragma unroll
    for (int hh = 0; hh < GH; ++hh) {
      float l = l_run[hh];
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
#pragma unroll
      for (int f = 0; f < NVF; ++f) *reinterpret_cast<f32x4*>(rec + (((w * GH + hh) * NVF + f) * 64 + lane) * 4) = oacc[hh][f];
      *reinterpret_cast<float2*>(ml + ((w * GH + hh) * 64 + lane) * 2) = make_float2(m_run[hh], l);
    }
    return;
  }
  if (!active || n >= nq) return;
#pragma unroll
  for (int hh = 0; hh < GH; ++hh) {
    float l = l_run[hh];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const float inv = 1.f / l;
#pragma unroll
    for (int f = 0; f < NVF; ++f) {
      union { uint16_t s[4]; u32x2 v; } o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o.s[i] = f32_to_f16_sat(oacc[hh][f][i] * inv);
      *reinterpret_cast<u32x2*>(op + packed_p_offset(row0 + n, (h0 + hh) * HD + f * 16 + g * 4, QD >> 4)) = o.v;
    }
  }
}

// Combines the key ranges of a tile, in key order: one workgroup per (tile, kv head and head group, query head of the
// wavefront, half of the head's dims), lanes as in the attention kernel.
template <int HD, int GH, int HG>
__global__ __launch_bounds__(256 * HG) void prefill_attn_merge_kernel(const int32_t* __restrict__ q_lens, const int32_t* __restrict__ seq_lens,
                                                                      int Hq, int Hkv, int G, const int32_t* __restrict__ tile_seq,
                                                                      const int32_t* __restrict__ tile_q0, const int32_t* __restrict__ meta,
                                                                      const int32_t* __restrict__ cum_rows, uint16_t* __restrict__ op,
                                                                      int max_tiles, int max_splits, const float* __restrict__ part) {
  constexpr int NVF = HD / 16, NF = NVF / 2;
  const int tile = blockIdx.x, jh = blockIdx.y, hh = blockIdx.z >> 1, f0 = (blockIdx.z & 1) * NF;
  if (tile >= meta[0]) return;
  const int b = tile_seq[tile], tq0 = tile_q0[tile], qlen = q_lens[b];
  const int prefix = seq_lens[b] - qlen;
  const int nsplit = pattn_splits((prefix + min(qlen, tq0 + 64) + 31) / 32, max_splits);
  if (nsplit <= 1) return;
  const int tid = threadIdx.x, w = tid >> 6, wave = w & 3, lane = tid & 63, n = lane & 15, g = lane >> 4;
  if (tq0 + wave * 16 + n >= qlen) return;
  const int head = (jh % Hkv) * G + ((jh / Hkv) * HG + (w >> 2)) * GH + hh;
  const float* rec0 = part + (int64_t)(jh * max_tiles + tile) * max_splits * pattn_record(HD, GH, HG);
  const int o_at = (((w * GH + hh) * NVF + f0) * 64 + lane) * 4, ml_at = 4 * HG * GH * 64 * (HD / 4) + ((w * GH + hh) * 64 + lane) * 2;
  float M = NEG_INF, L = 0.f;
  f32x4 o[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nsplit; s0 += 4) {  // four ranges per memory round trip
    float2 ml[4];
    f32x4 v[4][NF];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* rec = rec0 + (int64_t)min(s0 + u, nsplit - 1) * pattn_record(HD, GH, HG);
      ml[u] = *reinterpret_cast<const float2*>(rec + ml_at);
#pragma unroll
      for (int f = 0; f < NF; ++f) v[u][f] = *reinterpret_cast<const f32x4*>(rec + o_at + f * 256);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= nsplit) break;
      const float Mn = fmaxf(M, ml[u].x), ref = Mn == NEG_INF ? 0.f : Mn;
      const float a = __builtin_amdgcn_exp2f(M - ref), c = __builtin_amdgcn_exp2f(ml[u].x - ref);
      L = L * a + ml[u].y * c;
#pragma unroll
      for (int f = 0; f < NF; ++f) o[f] = o[f] * a + v[u][f] * c;
      M = Mn;
    }
  }
  const float inv = 1.f / L;
  const int64_t row = (int64_t)cum_rows[b] + tq0 + wave * 16 + n;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    union { uint16_t s[4]; u32x2 v; } out;
#pragma unroll
    for (int i = 0; i < 4; ++i) out.s[i] = f32_to_f16_sat(o[f][i] * inv);
    *reinterpret_cast<u32x2*>(op + packed_p_offset(row, head * HD + (f0 + f) * 16 + g * 4, (Hq * HD) >> 4)) = out.v;
  }
}

// ------------------------------------------------------------------------------------------------
// Host side

// Which kernel a prefill GEMM of T tokens, NRG row groups and KB k blocks uses: tb = 0: 256 x 256 tiles, 3: 256 rows x 192 tokens,
// 1 and 2: tiles of 128 rows x 128 tb tokens whose k range is shared by ks workgroups.  The choice is the least of the times in us that a
// fit of all kernels gives: rounds of one workgroup per compute unit, a time per k block, a fixed time per round
// (fill and epilogue) and, for a split range, the hand-over, whose last workgroup reads ks partial tiles.  Large calls
// keep the 256 x 256 tiles, which read least per product; small ones would leave most compute units idle with them.
// Measured at the 8B shape (us, 256 x 256 tiles against the choice): 333 tokens QKV 100 / 41 (128 tokens, no split), O 91 /
// 28 (128, 2 splits), gate/up 93 / 78 (192), down 256 / 59 (256 tokens, 4 splits); 1024 tokens 106 / 67, 93 / 44,
// 195 / 195, 261 / 117; 2048 tokens O 108 / 71, down 282 / 204; 8192 tokens: always 256 x 256 (gate/up 1388, the others 1660
// and 2030).
struct PGemmChoice { int tb, ks; float us; };
static PGemmChoice choose_pgemm(int T, int NRG, int KB) {
  constexpr int CUS = 256;
  const float per_kb[4] = {0.76f, 0.29f, 0.43f, 0.60f}, per_round[4] = {12.f, 5.f, 8.f, 11.f}, hand0[3] = {0.f, 7.f, 9.f}, hand1[3] = {0.f, 1.4f, 3.f};
  PGemmChoice best = {0, 1, 0.f};
  for (int tb = 0; tb <= 3; ++tb) {
    const int rows = tb % 3 ? 8 : 16, tokens = tb == 3 ? 192 : tb ? 128 * tb : 256;
    const int64_t tiles = (int64_t)((T + tokens - 1) / tokens) * ((NRG + rows - 1) / rows);
    for (int ks = 1; ks <= 8; ++ks) {
      if (ks > 1 && (tb % 3 == 0 || tiles * ks > CUS || KB < 8 * ks)) break;  // (parked tiles and counters are sized by this line)
      const float us = (float)((tiles * ks + CUS - 1) / CUS) * (per_kb[tb] * (float)((KB + ks - 1) / ks) + per_round[tb]) +
                       (ks > 1 ? hand0[tb] + hand1[tb] * ks : 0.f);
      if ((!tb && ks == 1) || us < best.us) best = {tb, ks, us};
    }
  }
  return best;
}

// bytes of parked partial tiles the splits of any call of up to maxT tokens need
uint64_t prefill_partial_bytes(int maxT, int NRG, int KB) {
  uint64_t most = 0;
  for (int64_t T = 128; T < (int64_t)maxT + 128; T += 128) {
    const PGemmChoice c = choose_pgemm((int)T, NRG, KB);
    if (c.ks > 1) {
      const uint64_t tiles = (uint64_t)((T + 128 * c.tb - 1) / (128 * c.tb)) * ((NRG + 7) / 8);
      if (tiles * c.ks * c.tb * 65536 > most) most = tiles * c.ks * c.tb * 65536;
    }
    if ((T / 256) * ((NRG + 7) / 8) > 256) break;  // more tiles than compute units from here on: never split
  }
  return most;
}

// rows of X of a call whose last positions ride along
int prefill_rows(int T, int batch) { return (T + 31) / 32 * 32 + (batch + 15) / 16 * 32; }

// Do the last positions of a call ride along as rows of its GEMMs?  Where that costs less, by the fit above, than the four
// products of the decode pass, which stream their weights at about 6 TB/s and take about 3 us, and 0.16 us per sequence, besides.
// One decision for all four products of a layer: calls whose tokens fill their tiles exactly would open another round of them and keep
// the pass (8B shape, one prompt: 333, 640, 768, 1500 and 3000 tokens ride, 512, 1024, 2048, 4096 and 8192 do not).
// Not for models with two weight planes, whose prefill reads the first alone.
bool prefill_rides(const www_model* m, int T, int batch) {
  if (m->wsplit || m->L < 2) return false;
  const float per_weight = m->int4_group ? 0.5f + 2.f / 32 : m->fp8 ? 1.f : 2.f;
  const int N[4] = {m->QKVN, m->d, 2 * m->F, m->d}, K[4] = {m->d, m->QD, m->d, m->Fp};
  float saved = 0.f, added = 0.f;
  for (int i = 0; i < 4; ++i) {
    saved += (float)N[i] * (float)K[i] * per_weight / 6e6f + 3.f + 0.16f * (float)batch;
    added += choose_pgemm(prefill_rows(T, batch), N[i] / 16, K[i] / 32).us - choose_pgemm(T, N[i] / 16, K[i] / 32).us;
  }
  return added < saved;
}

// Kernel (2: prefill_gemm_kernel, 3: prefill_gemm_small_kernel), tokens and rows per tile and k splits of GEMM `which` (0 QKV, 1 O,
// 2 gate/up, 3 down) of a prefill call, and whether its last positions ride along
void prefill_route(const www_model* m, int which, int T, int batch, int32_t out[5]) {
  const int N[4] = {m->QKVN, m->d, 2 * m->F, m->d}, K[4] = {m->d, m->QD, m->d, m->Fp};
  const bool rides = prefill_rides(m, T, batch);
  const PGemmChoice c = choose_pgemm(rides ? prefill_rows(T, batch) : T, N[which] / 16, K[which] / 32);
  const bool small = c.tb == 1 || c.tb == 2;
  out[0] = small ? 3 : 2; out[1] = c.tb == 0 ? 256 : c.tb == 3 ? 192 : 128 * c.tb; out[2] = small ? 128 : 256; out[3] = c.ks; out[4] = rides;
}

// Announces the GEMM kernels, which use more than 64 KiB of dynamic LDS, to the current device (when a model is loaded there).
// The residual GEMMs of large tiles always run the kernel that can carry last positions: their 256 x 256 epilogue spills 4 registers
// there and 63 without (8B shape, calls of 16 000 tokens: the two of a layer 2 x 1407 against 2 x 1467 us).  Not those of smaller tiles
// (8B shape, 512 tokens, down projection 76.0 us with it against 74.7; 1B shape, 1024 tokens, 49.2 against 47.6).
constexpr bool large_tiles_last(int epi, bool last) { return last || epi == PEPI_RESID; }
template <int EPI, bool QKN, bool LAST>
static hipError_t allow_pgemm_lds() {
  constexpr bool LL = large_tiles_last(EPI, LAST);
  auto allow = [](const void* kernel, int bytes) { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); };
  hipError_t e = allow(reinterpret_cast<const void*>(&prefill_gemm_kernel<EPI, QKN, LL, 4>), LL ? PGEMM_LAST_LDS_BYTES : PGEMM_LDS_BYTES);
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&prefill_gemm_kernel<EPI, QKN, LL, 3>), LL ? PGEMM_LAST_LDS_BYTES : PGEMM_LDS_BYTES);
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&prefill_gemm_small_kernel<EPI, QKN, 1, LAST>), PSG_LDS_BYTES);
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&prefill_gemm_small_kernel<EPI, QKN, 2, LAST>), PSG_LDS_BYTES);
  return e;
}
template <bool LAST>
static hipError_t allow_all_pgemm_lds() {
  hipError_t e = allow_pgemm_lds<PEPI_QKV, false, LAST>();
  if (e == hipSuccess) e = allow_pgemm_lds<PEPI_QKV, true, LAST>();
  if (e == hipSuccess) e = allow_pgemm_lds<PEPI_RESID, false, LAST>();
  if (e == hipSuccess) e = allow_pgemm_lds<PEPI_SWIGLU, false, LAST>();
  return e;
}
hipError_t prefill_allow_lds() {
  const hipError_t e = allow_all_pgemm_lds<false>();
  return e == hipSuccess ? allow_all_pgemm_lds<true>() : e;
}

// returns the number of entries per token a residual epilogue wrote into the sum-of-squares table
template <int EPI, bool QKN, bool LAST>
static int launch_pgemm_as(www_model* m, PGemmP& p, hipStream_t st) {
  p.n_tt = (p.T + 255) / 256;
  p.n_rt = (p.NRG + 15) / 16;
  if (p.wfactor == 0.f) p.wfactor = 1.f;  // not set: an unscaled matrix
  const PGemmChoice c = choose_pgemm(p.T, p.NRG, p.KB);
  if (c.tb % 3 == 0) {
    constexpr bool LL = large_tiles_last(EPI, LAST);
    if (c.tb == 3) p.n_tt = (p.T + 191) / 192;
    const dim3 grid(p.n_tt * p.n_rt);
    if (c.tb == 0) hipLaunchKernelGGL((prefill_gemm_kernel<EPI, QKN, LL, 4>), grid, dim3(256), LL ? PGEMM_LAST_LDS_BYTES : PGEMM_LDS_BYTES, st, p);
    else hipLaunchKernelGGL((prefill_gemm_kernel<EPI, QKN, LL, 3>), grid, dim3(256), LL ? PGEMM_LAST_LDS_BYTES : PGEMM_LDS_BYTES, st, p);
    return p.n_rt;
  }
  p.n_ttS = (p.T + 128 * c.tb - 1) / (128 * c.tb);
  p.n_rt128 = (p.NRG + 7) / 8;
  p.kb_per_split = (p.KB + c.ks - 1) / c.ks;
  p.ksplit = (p.KB + p.kb_per_split - 1) / p.kb_per_split;
  p.partial = m->partial; p.counters = m->counters; p.fence_handover = m->handover_fence; p.fault_flag = m->fault_dev;
  const dim3 grid(8 * ((p.n_rt128 + 7) / 8) * p.ksplit * p.n_ttS);
  if (c.tb == 1) hipLaunchKernelGGL((prefill_gemm_small_kernel<EPI, QKN, 1, LAST>), grid, dim3(256), PSG_LDS_BYTES, st, p);
  else hipLaunchKernelGGL((prefill_gemm_small_kernel<EPI, QKN, 2, LAST>), grid, dim3(256), PSG_LDS_BYTES, st, p);
  return p.n_rt128;
}
template <int EPI>
static int launch_pgemm(www_model* m, PGemmP& p, hipStream_t st) {
  if constexpr (EPI == PEPI_QKV) {
    if (p.qk_gain) return p.n_last ? launch_pgemm_as<EPI, true, true>(m, p, st) : launch_pgemm_as<EPI, true, false>(m, p, st);
  }
  return p.n_last ? launch_pgemm_as<EPI, false, true>(m, p, st) : launch_pgemm_as<EPI, false, false>(m, p, st);
}

// Shape of the attention workgroups: two query heads per wavefront pass, since their accumulators and operands fit 256
// registers, so two workgroups share a compute unit and one hides the other's softmax and LDS latencies (four heads per
// pass at one workgroup per unit: 1.5x slower).  With 128-wide heads two such head groups form one workgroup of eight
// wavefronts (still two per SIMD) and share the copy of the keys and values into LDS, which halves the code-to-fp16
// conversions per query head.  max_splits: most key ranges per tile, for up to two workgroups per compute unit (half of the
// tiles the host has to provide for are usually empty or short; limits of 128, 256 and 512 workgroups: 16 sequences of 16 -
// 32 tokens over mixed prefixes 13.0, 12.6, 12.6 ms, 4 x 512 over 2000 33.4, 33.3, 34.4, one prompt of 2000 32.1, 32.4, 32.6).
struct PAttnShape { int GH, HG, items, max_splits; };
static PAttnShape pattn_shape(int hd, int Hkv, int G, int max_tiles, int max_pos) {
  PAttnShape a;
  a.GH = (G % 2 == 0) ? 2 : 1;
  a.HG = (hd == 128 && (G / a.GH) % 2 == 0) ? 2 : 1;
  a.items = max_tiles * Hkv * (G / a.GH / a.HG);
  a.max_splits = a.items <= PATTN_MAX_ITEMS ? 2 * PATTN_MAX_ITEMS / a.items : 1;
  if (a.max_splits > 16) a.max_splits = 16;
  a.max_splits = pattn_splits((max_pos + 31) / 32, a.max_splits);
  return a;
}

// bytes of parked softmax states any call needs
uint64_t prefill_attn_part_bytes(int hd, int Hkv, int G, int maxT, int maxB, int max_pos) {
  uint64_t most = 0;
  for (int tiles = 1; tiles <= maxT / ATTN_TQ + maxB; ++tiles) {
    const PAttnShape a = pattn_shape(hd, Hkv, G, tiles, max_pos);
    if (a.items > PATTN_MAX_ITEMS) break;
    const uint64_t bytes = a.max_splits > 1 ? (uint64_t)a.items * a.max_splits * pattn_record(hd, a.GH, a.HG) * 4 : 0;
    if (bytes > most) most = bytes;
  }
  return most;
}

template <int HD>
static void launch_pattn(www_model* m, const uint16_t* kplane, const uint16_t* vplane, const float* kvscale, const int32_t* qlens, const int32_t* lens,
                         const int32_t* table, int max_tiles, hipStream_t st) {
  const PAttnShape a = pattn_shape(HD, m->Hkv, m->G, max_tiles, m->max_pos);
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
  const int32_t* cum_rows = m->meta + 16;
#define PATTN(GH_, HG_)                                                                                                            \
  {                                                                                                                                \
    hipLaunchKernelGGL((prefill_attn_kernel<HD, GH_, HG_>), dim3(a.items * a.max_splits), dim3(256 * HG_), 0, st,                  \
                       (const uint16_t*)m->qp, kplane, vplane, kvscale, qlens, lens, table, (int)m->cfg.max_blocks_per_seq, m->Hq, \
                       m->Hkv, m->G, m->tile_seq, m->tile_q0, m->meta, cum_rows, scale_log2, (uint16_t*)m->op, max_tiles,          \
                       a.max_splits, m->partial);                                                                                  \
    if (a.max_splits > 1)                                                                                                          \
      hipLaunchKernelGGL((prefill_attn_merge_kernel<HD, GH_, HG_>), dim3(max_tiles, m->Hkv * (m->G / GH_ / HG_), GH_ * 2),         \
                         dim3(256 * HG_), 0, st, qlens, lens, m->Hq, m->Hkv, m->G, m->tile_seq, m->tile_q0, m->meta, cum_rows,     \
                         (uint16_t*)m->op, max_tiles, a.max_splits, m->partial);                                                   \
  }
  if constexpr (HD == 128) {
    if (a.HG == 2) { PATTN(2, 2) return; }
  }
  if (a.GH == 2) PATTN(2, 1) else PATTN(1, 1)
#undef PATTN
}

int run_prefill(www_model* m, const int32_t* tok, const int32_t* qlens, const int32_t* lens, const int32_t* table, int batch, int T,
                bool rides, hipStream_t st) {
  const int d = m->d;
  int32_t* cum = m->meta + 16;
  const int first_last = rides ? (T + 31) / 32 * 32 : 0, n_last = rides ? batch : 0, rows = rides ? prefill_rows(T, batch) : T;
  hipLaunchKernelGGL(prefill_meta_kernel, dim3(1), dim3(1024), 0, st, tok, qlens, lens, batch, T, m->row_seq, m->row_pos, m->tile_seq,
                     m->tile_q0, m->meta, m->last_tok, cum, first_last, rows);
  if (rides) launch_attn_plan(m, lens, batch, st);
  if (m->cfg.weight_dtype == WWW_DTYPE_F32)
    hipLaunchKernelGGL(embed_rows_kernel<float>, dim3(T + n_last), dim3(256), 0, st, tok, (const float*)m->embed, d, m->layers[0].attn_norm, m->hp,
                       (uint16_t*)m->xn, m->ssq_p, T, first_last, m->last_tok, m->h);
  else
    hipLaunchKernelGGL(embed_rows_kernel<uint16_t>, dim3(T + n_last), dim3(256), 0, st, tok, (const uint16_t*)m->embed, d, m->layers[0].attn_norm,
                       m->hp, (uint16_t*)m->xn, m->ssq_p, T, first_last, m->last_tok, m->h);
  int n_ssq = 1;
  const int max_tiles = T / ATTN_TQ + batch;
  auto gemm = [&]() {
    PGemmP p = {};
    p.T = rows; p.T_new = T; p.first_last = rides ? first_last : 0x7fffffff; p.n_last = n_last; p.h_last = m->h;
    return p;
  };
  for (int l = 0; l < m->L; ++l) {
    const LayerW& w = m->layers[l];
    uint16_t* kplane = (uint16_t*)m->kv + (int64_t)(2 * l) * m->kv_plane;
    uint16_t* vplane = (uint16_t*)m->kv + (int64_t)(2 * l + 1) * m->kv_plane;
    float* kvscale = m->kv_scales + (int64_t)l * m->kv_scale_plane;
    {
      PGemmP p = gemm();
      p.W = (const u32x4*)w.wqkv; p.wfactor = w.sqkv; p.NRG = m->QKVN / 16; p.KB = d / 32; p.X = (const u32x4*)m->xn;
      p.ssq_in = m->ssq_p; p.n_ssq_in = n_ssq; p.inv_dim = 1.f / d; p.eps = m->cfg.rms_eps;
      p.qp = (uint16_t*)m->qp; p.kplane = kplane; p.vplane = vplane; p.kvscale = kvscale; p.row_seq = m->row_seq; p.row_pos = m->row_pos; p.table = table;
      p.mbs = m->cfg.max_blocks_per_seq; p.hd = m->hd; p.Hq = m->Hq; p.Hkv = m->Hkv; p.rope = m->rope; p.qk_gain = w.qk_gain;
      p.q_hi = m->q_hi; p.q_lo = m->q_lo; p.qscale = 1.4426950408889634f / sqrtf((float)m->hd);
      launch_pgemm<PEPI_QKV>(m, p, st);
    }
    if (l == m->L - 1) break;  // only this layer's keys and values (and the last positions' queries) are still needed
    if (rides) launch_decode_attn(m, l, lens, table, batch, (uint16_t*)m->op, 0, first_last, st);
    if (m->hd == 128) launch_pattn<128>(m, kplane, vplane, kvscale, qlens, lens, table, max_tiles, st);
    else launch_pattn<64>(m, kplane, vplane, kvscale, qlens, lens, table, max_tiles, st);
    {
      PGemmP p = gemm();
      p.W = (const u32x4*)w.wo; p.wfactor = w.so; p.NRG = d / 16; p.KB = m->QD / 32; p.X = (const u32x4*)m->op;
      p.hp = m->hp; p.d = d; p.gain_next = w.ffn_norm; p.xn_out = (uint16_t*)m->xn; p.ssq_out = m->ssq_p;
      n_ssq = launch_pgemm<PEPI_RESID>(m, p, st);
    }
    {
      PGemmP p = gemm();
      p.W = (const u32x4*)w.wgu; p.wfactor = w.sgu; p.NRG = 2 * m->F / 16; p.KB = d / 32; p.X = (const u32x4*)m->xn;
      p.ssq_in = m->ssq_p; p.n_ssq_in = n_ssq; p.inv_dim = 1.f / d; p.eps = m->cfg.rms_eps;
      p.ap = (uint16_t*)m->ap; p.Fp = m->Fp;
      launch_pgemm<PEPI_SWIGLU>(m, p, st);
    }
    {
      PGemmP p = gemm();
      p.W = (const u32x4*)w.wd; p.wfactor = w.sd; p.NRG = d / 16; p.KB = m->Fp / 32; p.X = (const u32x4*)m->ap;
      p.hp = m->hp; p.d = d; p.gain_next = m->layers[l + 1].attn_norm; p.xn_out = (uint16_t*)m->xn; p.ssq_out = m->ssq_p;
      n_ssq = launch_pgemm<PEPI_RESID>(m, p, st);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("prefill launch failed: %s", hipGetErrorString(e));
    return WWW_E_HIP;
  }
  return WWW_OK;
}

// Host-side view of the prefill GEMM's workgroup -> tile map (tests).
extern "C" __attribute__((visibility("default"))) int www_debug_prefill_tile(int32_t workgroup, int32_t token_tiles, int32_t row_tiles, int32_t* token_tile_out,
                                      int32_t* row_tile_out) {
  if (!token_tile_out || !row_tile_out || token_tiles < 1 || row_tiles < 1 || workgroup < 0 ||
      (int64_t)workgroup >= (int64_t)token_tiles * row_tiles || (int64_t)token_tiles * row_tiles > 0x7fffffff) {
    set_error("www_debug_prefill_tile: arguments out of range");
    return WWW_E_INVALID_ARG;
  }
  int tt, rt;
  pgemm_tile_of(workgroup, token_tiles, row_tiles, &tt, &rt);
  *token_tile_out = tt;
  *row_tile_out = rt;
  return WWW_OK;
}
