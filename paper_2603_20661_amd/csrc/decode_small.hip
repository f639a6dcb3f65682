// Decode GEMMs for up to 32 tokens: Y^T[n][t] = sum_k W[n][k] X[t][k] with the epilogues of the decode path.
#include <math.h>

#include "decode_gemm.h"

// A workgroup owns 16 R RW rows and a range of k, which it cuts over its eight wavefronts: wavefront (rw, kw) takes R row
// groups and every KW-th chunk of KC k blocks and loads weights and activations straight into registers, D chunks ahead; no
// LDS and no barrier in the loop.  The partial tiles are added through LDS in wavefront order.
//
// What bounds it: the weight stream (6.2 TB/s at best) or what a compute unit takes in (about 52 KB per us, weights and
// activations together), plus launch, first round trip and the sum at the end, about 4 us.  In skinny_gemm_kernel a
// workgroup has 128 rows, so a narrow GEMM needs many k splits, whose tiles meet in memory (three dependent round trips and
// ksplit tiles read by one workgroup), and four wavefronts with one chunk in flight each wait for every chunk.  With few
// tokens the activations are small, so a workgroup can own few rows and a long k range instead.
// XF: fragments of activations per k block.  1: up to 8 tokens, the hi parts are the columns 0 .. 7 and the lo parts the
// columns 8 .. 15 of one fragment (half the products and half the loads); 2: up to 16 tokens, hi and lo; 4: up to 32.
constexpr int SG_NW = 8;
constexpr int sg_kc(int wmode, int XF) { return XF == 4 && wmode != WMODE_INT4 ? 2 : 4; }
// registers of one chunk
constexpr int sg_set(int wmode, int R, int XF) {
  return sg_kc(wmode, XF) * (R * (wmode == WMODE_F16 ? 4 : wmode == WMODE_SPLIT ? 8 : 2) + 4 * XF) - (wmode == WMODE_INT4 ? 2 * R : 0);
}
// four wavefronts per SIMD (128 registers) where two chunks fit, two otherwise
constexpr int sg_eu(int wmode, int R, int XF) { return sg_set(wmode, R, XF) + 4 * R * (XF / 4) <= 40 ? 4 : 2; }
constexpr int sg_depth(int wmode, int R, int XF) {
  const int set = sg_set(wmode, R, XF), d = (sg_eu(wmode, R, XF) == 4 ? 88 : 150) / set;
  return d > 4 ? 4 : d < 2 ? 2 : d;
}

template <int WMODE, int EPI, int R, int RW, int XF>
__global__ __launch_bounds__(64 * SG_NW, sg_eu(WMODE, R, XF)) void small_gemm_kernel(const GemmP p) {
  constexpr bool WSPLIT = WMODE == WMODE_SPLIT, W8 = WMODE == WMODE_FP8, W4 = WMODE == WMODE_INT4;
  constexpr int D = sg_depth(WMODE, R, XF), KC = sg_kc(WMODE, XF), KW = SG_NW / RW, RT = R * RW, TB = XF == 4 ? 2 : 1;
  static_assert(EPI != EPI_SWIGLU || R % 2 == 0, "a gate row group sits in front of its up row group");
  static_assert(EPI == EPI_LOGITS || RT <= SG_NW, "one wavefront per row group in the epilogue");
  __shared__ f32x4 red[KW][RT][TB][64];
  __shared__ float s_scale[16 * TB];
  __shared__ float s_head[2][8][16 * TB];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kw = wave % KW, rw = wave / KW;

  // Workgroup id -> work item.  Workgroups that hand partial results over (the k splits of a row tile; in the QKV GEMM also
  // the row tiles of a head) form a group; the members of a group get ids that are equal modulo 8, so they run behind one L2.
  // The key and value heads, which always end with a hand-over, come first.
  const int slot = blockIdx.x >> 3, within = slot % p.zbs;
  const int g0 = (blockIdx.x & 7) + 8 * (slot / p.zbs);
  if (g0 >= p.row_tiles) return;  // grid padding when the groups are not a multiple of 8
  const int group = EPI == EPI_QKV ? p.row_tiles - 1 - g0 : g0;
  const int split = within % p.ksplit, member = within / p.ksplit;
  const int hrg = EPI == EPI_QKV ? p.hd >> 4 : RT;  // row groups of a group
  const int rg0 = group * hrg + member * RT;
  const int kb_begin = split * p.kb_per_split, nkb = min(p.KB, kb_begin + p.kb_per_split) - kb_begin;
  const int nch = (nkb + KC - 1) / KC;
  const int n_w = (nch - kw + KW - 1) / KW;  // chunks of this wavefront (none: it only helps with the rest)
  // do results of other workgroups enter the epilogue?
  const bool handover = (EPI == EPI_QKV || EPI == EPI_RESID) && (p.ksplit > 1 || (EPI == EPI_QKV && p.zbs > 1 && (group >= p.Hq || p.qk_gain)));

  // token of this lane's accumulators (XF == 1: of the sum of its hi and lo columns)
  const int tsub = lane & 15, rsub = (lane >> 4) * 4;
  const int tlow = XF == 1 ? lane & 7 : tsub;
  // row group this wavefront finishes (SWIGLU: the gate's, its up rows are the next)
  const int fin = EPI == EPI_SWIGLU ? 2 * wave : wave;
  const int n_fin = EPI == EPI_SWIGLU ? RT / 2 : handover ? hrg : RT;
  const int frg = (handover && EPI == EPI_QKV ? group * hrg : rg0) + fin, frgc = min(frg, p.NRG - 1);
  const int n0 = frgc * 16 + rsub;

  // Operands of the epilogue are requested first; they have arrived when the first weights have.  A token's sums of squares
  // are read by 32 / TB threads, two (four) 16-byte pieces each, which covers d_model = 4096.
  constexpr int SUB = 32 / TB, NSQ = 2 * TB;
  f32x4 sq[NSQ];
  const int sq_tok = tid / SUB, sq_sub = tid % SUB;
  const float* sq_row = p.ssq_in + (int64_t)min(sq_tok, p.M - 1) * SSQ_ROWS;
  if (p.ssq_in) {
#pragma unroll
    for (int i = 0; i < NSQ; ++i) sq[i] = *reinterpret_cast<const f32x4*>(sq_row + (i * SUB + sq_sub) * 4);
  }
  int tok[TB], pos[TB], blk[TB];
  f32x4 hv[TB], gv, cs[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    tok[tb] = min(tb * 16 + tlow, p.M - 1);
    if constexpr (EPI == EPI_QKV) pos[tb] = p.seq_lens[tok[tb]] - 1;
    if constexpr (EPI == EPI_RESID) hv[tb] = *reinterpret_cast<const f32x4*>(p.h + (int64_t)tok[tb] * p.d + n0);
  }
  if constexpr (EPI == EPI_QKV) {
    if (p.qk_gain) gv = *reinterpret_cast<const f32x4*>(p.qk_gain + (n0 / p.hd < p.Hq ? 0 : p.hd) + n0 % p.hd);
  }
  if constexpr (EPI == EPI_RESID) gv = *reinterpret_cast<const f32x4*>(p.gain_next + n0);

  struct Set {
    u32x4 w[W4 ? 1 : W8 ? KC / 2 : WSPLIT ? 2 * KC : KC][R];
    u32x2 sc[R];
    u32x4 x[KC][XF];
  };
  // columns without a token read the last one's lines again
  const int xl = XF == 1 ? ((lane >> 3) & 1) * 64 + (lane & 48) + min(lane & 7, p.M - 1) : (lane & 48) + min(tsub, min(p.M, 16) - 1);
  const int xl2 = XF == 4 ? 128 + (lane & 48) + min(tsub, p.M - 17) : 0;  // the second group of 16 tokens
  int rgc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) rgc[r] = min(rg0 + rw * R + r, p.NRG - 1);
  // (loads past the end of the k range are redirected to its last valid block, their products are skipped)
  auto load = [&](Set& s, int i) __attribute__((always_inline)) {
    const int kb0 = kb_begin + (kw + KW * i) * KC, last = kb_begin + nkb - 1;
    if constexpr (W4) {
      const int chunk = min(kb0 >> 2, last >> 2);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        s.w[0][r] = p.W[((int64_t)chunk * p.NRG + rgc[r]) * 64 + lane];
        s.sc[r] = p.Wscale[((int64_t)chunk * p.NRG + rgc[r]) * 16 + tsub];
      }
    } else if constexpr (W8) {
#pragma unroll
      for (int j = 0; j < KC / 2; ++j) {
        const int pair = min((kb0 >> 1) + j, last >> 1);
#pragma unroll
        for (int r = 0; r < R; ++r) s.w[j][r] = p.W[((int64_t)pair * p.NRG + rgc[r]) * 64 + lane];
      }
    } else {
#pragma unroll
      for (int j = 0; j < KC; ++j) {
        const int64_t kb = min(kb0 + j, last);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          s.w[j][r] = p.W[(kb * p.NRG + rgc[r]) * 64 + lane];
          if constexpr (WSPLIT) s.w[KC + j][r] = p.Wlo[(kb * p.NRG + rgc[r]) * 64 + lane];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      const int64_t kb = min(kb0 + j, last);
#pragma unroll
      for (int f = 0; f < XF; ++f) s.x[j][f] = p.X[kb * (128 * TB) + (f & 1) * 64 + (f < 2 ? xl : xl2)];
    }
  };
  f32x4 acc[R][TB];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[r][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](Set& s, int nv) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      if (j >= nv) break;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        f16x8 a;
        if constexpr (W4) {
          const u32x4 raw = s.w[0][r];
          const uint32_t word = j == 0 ? raw.x : j == 1 ? raw.y : j == 2 ? raw.z : raw.w, s2 = j < 2 ? s.sc[r].x : s.sc[r].y;
          const uint32_t s16 = (j & 1) ? (s2 >> 16) : (s2 & 0xFFFFu);
          a = int4x8_to_f16x8(word, __builtin_bit_cast(f16x2, s16 | (s16 << 16)));
        } else if constexpr (W8) {
          const u32x4 raw = s.w[j >> 1][r];
          a = (j & 1) ? fp8x8_to_f16x8(raw.z, raw.w) : fp8x8_to_f16x8(raw.x, raw.y);
        } else {
          a = as_f16x8(s.w[j][r]);
        }
#pragma unroll
        for (int f = 0; f < XF; ++f) {
          f32x4& c = acc[r][f >> 1];
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, as_f16x8(s.x[j][f]), c, 0, 0, 0);
          if constexpr (WSPLIT)
            if ((f & 1) == 0) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(s.w[KC + j][r]), as_f16x8(s.x[j][f]), c, 0, 0, 0);
        }
      }
    }
  };
  auto valid = [&](int i) __attribute__((always_inline)) { return min(KC, nkb - (kw + KW * i) * KC); };

  Set set[D];
#pragma unroll
  for (int s = 0; s < D; ++s) load(set[s], s);  // (a wavefront with fewer chunks reads the last blocks again)
  __builtin_amdgcn_sched_barrier(0);
  if (p.ssq_in) {  // the threads of a token add its entries in a fixed order
    auto part = [&](f32x4 v, int e0) __attribute__((always_inline)) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) s += e0 + e < p.n_ssq_in ? v[e] : 0.f;
      return s;
    };
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NSQ; ++i) s += part(sq[i], (i * SUB + sq_sub) * 4);
    for (int i = NSQ; i * SUB * 4 < p.n_ssq_in; ++i) s += part(*reinterpret_cast<const f32x4*>(sq_row + (i * SUB + sq_sub) * 4), (i * SUB + sq_sub) * 4);
#pragma unroll
    for (int o = SUB / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (sq_sub == 0) s_scale[sq_tok] = rsqrtf(s * p.inv_dim + p.eps) * p.wfactor;
  } else if (tid < 16 * TB) {
    s_scale[tid] = p.wfactor;
  }
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      blk[tb] = kv_block_id(p.table + (int64_t)tok[tb] * p.mbs, pos[tb]);
      cs[tb] = *reinterpret_cast<const f32x4*>(p.rope + (int64_t)pos[tb] * (p.hd / 2) + ((n0 % p.hd) >> 1));
    }
  }
  int i = 0;
  for (; i + 2 * D <= n_w; i += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      compute(set[s], KC);
      load(set[s], i + s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < D; ++s) {
    if (i + s < n_w) compute(set[s], valid(i + s));
    if (i + s + D < n_w) load(set[s], i + s + D);
  }
#pragma unroll
  for (int s = 0; s < D - 1; ++s)
    if (i + s + D < n_w) compute(set[s], valid(i + s + D));

#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) red[kw][rw * R + r][tb][lane] = acc[r][tb];
  __syncthreads();
  auto sum = [&](int r, int tb) __attribute__((always_inline)) {
    f32x4 v = red[0][r][tb][lane];
#pragma unroll
    for (int w = 1; w < KW; ++w) v += red[w][r][tb][lane];
    if constexpr (XF == 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], 8);
    }
    return v;
  };
  auto valid_token = [&](int tb) __attribute__((always_inline)) { return tlow == tsub && tb * 16 + tlow < p.M; };

  if constexpr (EPI == EPI_LOGITS) {
    float best[TB];
    int best_at[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) { best[tb] = NEG_INF; best_at[tb] = 0x7fffffff; }
    for (int q = wave; q < RT; q += SG_NW) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        const f32x4 o = sum(q, tb) * s_scale[tb * 16 + tlow];
        const int n = (rg0 + q) * 16 + rsub;
        if (valid_token(tb) && rg0 + q < p.NRG) {
          *reinterpret_cast<f32x4*>(p.logits + (int64_t)(tb * 16 + tlow) * p.V + n) = o;
#pragma unroll
          for (int e = 0; e < 4; ++e) argmax_take(best[tb], best_at[tb], o[e], n + e);
        }
      }
    }
    if (!p.best_val) return;  // the largest of this workgroup per token, for argmax_kernel
    __shared__ float s_best[SG_NW][16 * TB];
    __shared__ int s_at[SG_NW][16 * TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      argmax_of_rows(best[tb], best_at[tb]);
      if (lane < 16) { s_best[wave][tb * 16 + lane] = best[tb]; s_at[wave][tb * 16 + lane] = best_at[tb]; }
    }
    __syncthreads();
    if (tid < 16 * TB && tid < p.M) {
      float b = s_best[0][tid];
      int at = s_at[0][tid];
#pragma unroll
      for (int w = 1; w < SG_NW; ++w) argmax_take(b, at, s_best[w][tid], s_at[w][tid]);
      p.best_val[(int64_t)tid * p.row_tiles + group] = b;
      p.best_idx[(int64_t)tid * p.row_tiles + group] = at;
    }
    return;
  }
  f32x4 v[TB], up[TB];
  if (wave < (EPI == EPI_SWIGLU ? RT / 2 : RT)) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      v[tb] = sum(fin, tb);
      if constexpr (EPI == EPI_SWIGLU) up[tb] = sum(fin + 1, tb);
    }
  }
  if constexpr (EPI == EPI_QKV || EPI == EPI_RESID) {
    if (handover) {
      // parked as [split][row group][tb][lane]; the workgroup of the group that comes last adds the splits in order
      const __amdgpu_buffer_rsrc_t prs = shared_rsrc(p.partial);
      auto unit = [&](int sp, int rg, int tb) __attribute__((always_inline)) { return (uint32_t)(((sp * p.NRG + rg) * TB + tb) * 64 + lane) * 16u; };
      if (wave < RT && rg0 + wave < p.NRG) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) store_shared_f32x4(prs, unit(split, rg0 + wave, tb), v[tb]);
      }
      wait_own_memory_ops();
      __syncthreads();
      if (tid == 0) s_last = arrive_last(&p.counters[group], p.zbs, p.fence_handover, p.fault_flag);
      __syncthreads();
      if (!s_last) return;
      // the fenced hand-over's other half (acquire side of the producers' release fences)
      if (p.fence_handover) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (tid == 0) __hip_atomic_store(&p.counters[group], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (wave < n_fin) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) v[tb] = f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 pv[4][TB];
        add_in_order<4>(p.ksplit,
            [&](int u, int sp) __attribute__((always_inline)) {
#pragma unroll
              for (int tb = 0; tb < TB; ++tb) pv[u][tb] = load_shared_f32x4(prs, unit(sp, frgc, tb));
            },
            [&](int u) __attribute__((always_inline)) {
#pragma unroll
              for (int tb = 0; tb < TB; ++tb) v[tb] += pv[u][tb];
            });
      }
    }
  }
  if (wave >= n_fin) return;  // (the barriers below count the wavefronts that are left)
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const float scale = s_scale[tb * 16 + tlow];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[tb][e] *= scale;
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) up[tb][e] *= scale;
    }
  }
  if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      union { uint16_t s[4]; u32x2 v; } hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) split_f16(v[tb][e] / (1.f + __expf(-v[tb][e])) * up[tb][e], hi.s[e], lo.s[e]);
      if (valid_token(tb) && frg + 1 < p.NRG) {
        const int f0 = (frg >> 1) * 16 + rsub;
        *reinterpret_cast<u32x2*>(p.xa + packed_x_offset(f0, tb * 16 + tlow, TB, 0)) = hi.v;
        *reinterpret_cast<u32x2*>(p.xa + packed_x_offset(f0, tb * 16 + tlow, TB, 1)) = lo.v;
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int t = tb * 16 + tlow;
      float s = 0.f;
      union { uint16_t s[4]; u32x2 v; } hi, lo;
      f32x4 hn;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hn[e] = hv[tb][e] + v[tb][e];
        s += hn[e] * hn[e];
        split_f16(hn[e] * gv[e], hi.s[e], lo.s[e]);
      }
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (valid_token(tb) && frg < p.NRG) {
        *reinterpret_cast<f32x4*>(p.h + (int64_t)t * p.d + n0) = hn;
        *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, TB, 0)) = hi.v;
        *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, TB, 1)) = lo.v;
        if (lane < 16) p.ssq_out[(int64_t)t * SSQ_ROWS + frg] = s;  // one entry per row group
      }
    }
  } else if constexpr (EPI == EPI_QKV) {  // `group` is the head
    const bool rotated = group < p.Hq + p.Hkv;
    if (p.qk_gain) {  // 1 / rms of the head vector, its row groups added in order
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        float s = v[tb][0] * v[tb][0] + v[tb][1] * v[tb][1] + v[tb][2] * v[tb][2] + v[tb][3] * v[tb][3];
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < 16) s_head[0][wave][tb * 16 + lane] = s;
      }
      __syncthreads();
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        float tot = 0.f;
        for (int w = 0; w < n_fin; ++w) tot += s_head[0][w][tb * 16 + tsub];
        const float rs = rsqrtf(tot / (float)p.hd + p.eps);
        if (rotated) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[tb][e] *= rs * gv[e];
        }
      }
    }
    const int c0 = n0 % p.hd;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      if (rotated) {  // rows arrive with the rotary pair (i, i + hd/2) at neighbouring positions (2i, 2i+1)
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
          const float a = v[tb][2 * pr], b = v[tb][2 * pr + 1], c = cs[tb][2 * pr], s = cs[tb][2 * pr + 1];
          v[tb][2 * pr] = a * c - b * s;
          v[tb][2 * pr + 1] = b * c + a * s;
        }
      }
      if (group < p.Hq) {
        // queries leave as fp16 hi + lo, already multiplied by log2(e)/sqrt(hd), in the order the attention kernel loads them
        union { uint16_t s[4]; u32x2 v; } qh, ql;
#pragma unroll
        for (int e = 0; e < 4; ++e) split_f16(v[tb][e] * p.qscale, qh.s[e], ql.s[e]);
        if (valid_token(tb)) {
          *reinterpret_cast<u32x2*>(p.q_hi + (int64_t)(tb * 16 + tlow) * (p.Hq * p.hd) + n0) = qh.v;
          *reinterpret_cast<u32x2*>(p.q_lo + (int64_t)(tb * 16 + tlow) * (p.Hq * p.hd) + n0) = ql.v;
        }
      }
    }
    if (group < p.Hq) return;
    // keys and values go to the cache as 16-bit codes with the scale of their (token, head) vector
    float amax[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      float am = fmaxf(fmaxf(__builtin_fabsf(v[tb][0]), __builtin_fabsf(v[tb][1])), fmaxf(__builtin_fabsf(v[tb][2]), __builtin_fabsf(v[tb][3])));
      am = fmaxf(am, __shfl_xor(am, 16));
      am = fmaxf(am, __shfl_xor(am, 32));
      if (lane < 16) s_head[1][wave][tb * 16 + lane] = am;
      amax[tb] = am;
    }
    __syncthreads();
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      float am = amax[tb];
      for (int w = 0; w < n_fin; ++w) am = fmaxf(am, s_head[1][w][tb * 16 + tsub]);
      if (!valid_token(tb)) continue;
      const int64_t slot_id = kv_slot_in_block(blk[tb], pos[tb]), kblk = slot_id / KV_BS;
      const int at = (int)(slot_id % KV_BS);
      const bool is_v = !rotated;
      const int j = group - p.Hq - (is_v ? p.Hkv : 0);
      const float inv = kv_code_inv(am);
      union { uint16_t s[4]; u32x2 v; } code;
#pragma unroll
      for (int e = 0; e < 4; ++e) code.s[e] = kv_code(v[tb][e], inv);
      uint16_t* dst = (is_v ? p.vplane : p.kplane) + (kblk * p.Hkv + j) * (int64_t)(KV_BS * p.hd);
      if (!is_v) {
        *reinterpret_cast<u32x2*>(dst + k_cache_offset(at, c0)) = code.v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[v_cache_offset(at, c0 + e)] = code.s[e];
      }
      if (c0 == 0) p.kvscale[kv_scale_offset(kblk, p.Hkv, j) + (is_v ? 16 : 0) + at] = kv_code_scale(am);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Host side
// Rows and k splits of the QKV and residual GEMMs: the least of the times a model of two rates gives, the weight stream at
// 6.2 TB/s and the intake of a compute unit at 52 KB per us (its weights, and the activations of its k range), the shorter of
// the two hidden to three quarters behind the longer, plus 3 us and the reading of the parked tiles where results are handed
// over (4 us with split k ranges).  Many rows save activations, few rows or more splits keep every compute unit at work.
// 8B shape, us: down projection of FP8 weights, 16 tokens, 1 row group without splits 21.4, 2 x 2 splits 19.7, 4 x 4 16.6; O
// projection of fp16 weights, 1 token, 1 x 1 8.5, 2 x 2 9.8, 4 x 4 11.2; QKV, 16 tokens, FP8: 1 x 1 15.8, 2 x 1 14.5, 4 x 2 12.5.
// Where two workgroups fit a compute unit, a partial second round counts as its part from one and a half rounds on only: with less
// a few units that have two hold up all others (4 tokens, 320 row groups of 432 k blocks, 1 x 1: 38.7; the other kernel 31.8).
static SmallShape narrow_shape(int epi, int NRG, int KB, int hd, int xf, int wmode) {
  const float CUS = (float)decode_wg_target();
  const float wbytes = wmode == WMODE_INT4 ? 0.5f + 2.f / 32 : wmode == WMODE_FP8 ? 1.f : 2.f;
  const int chunk = SG_NW * sg_kc(wmode, xf);  // k blocks of one chunk of every wavefront: an unfilled round costs a whole one
  SmallShape best = {1, 1, xf, 1, (KB + 3) / 4 * 4, 0.f};
  for (int R = 1; R <= 4; R *= 2)
    for (int ks = 1; ks <= 8; ++ks) {
      const int per = ((KB + ks - 1) / ks + 3) / 4 * 4, members = epi == EPI_QKV ? hd / 16 / R : 1;
      if ((KB + per - 1) / per != ks || members < 1 || members * ks > 31) continue;  // (arrivals of a group: 5 bits per XCD)
      if (ks > 1 && (per < chunk || (NRG + R - 1) / R * ks > decode_wg_target())) break;
      const float groups = (float)((NRG + R - 1) / R) * (float)ks, fill = groups < CUS ? 1.f : groups / CUS;
      const float rounds = sg_eu(wmode, R, xf) == 4 && fill >= 1.5f ? fill : ceilf(fill);  // two workgroups share a compute unit, or one has it
      const float intake = rounds * (float)((per + chunk - 1) / chunk * chunk) * 32.f * (16.f * (float)R * wbytes + 32.f * (float)xf) / 52e3f;
      const float stream = (float)NRG * 16.f * (float)KB * 32.f * wbytes / 6.2e6f;
      const float us = (intake > stream ? intake + 0.25f * stream : stream + 0.25f * intake) + (ks > 1 ? 1.f : 0.f) + (members * ks > 1 ? 3.f + (float)(ks * R * (xf == 4 ? 2 : 1)) * 1024.f / 52e3f : 0.f);
      if ((R == 1 && ks == 1) || us < best.us) best = {R, 1, xf, ks, per, us};
    }
  return best;
}

// The same estimate for skinny_gemm_kernel: row tiles of 8 row groups, activations of whole groups of 16 tokens
static float general_us(int NRG, int KB, int M, float wbytes) {
  const int row_tiles = (NRG + 7) / 8, MT = M <= 16 ? 1 : 2, cus = decode_wg_target();
  int ks, per;
  choose_split(row_tiles, 1, KB, &ks, &per);
  const float intake = (float)((row_tiles * ks + cus - 1) / cus * per) * 32.f * (128.f * wbytes + 64.f * (float)MT) / 52e3f;
  const float stream = (float)NRG * 16.f * (float)KB * 32.f * wbytes / 6.2e6f;
  return (intake > stream ? intake + 0.25f * stream : stream + 0.25f * intake) + (ks > 1 ? 4.f + (float)(ks * 8 * MT) * 1024.f / 52e3f : 0.f);
}

// Which GEMMs of a step of M tokens run here (us per launch against skinny_gemm_kernel; 8B shape 1, 12, 24 sequences, 1B shape
// 4 and 32): QKV 13.5 / 15.5, 15.3 / 16.0, 17.7 / 17.9, 8.4 / 11.2, 11.7 / 13.9; O 8.5 / 12.3, 10.5 / 12.4, 11.6 / 14.1, 5.0 / 8.7,
// 8.0 / 10.0; down 22.4 / 25.8, 24.8 / 26.5, 26.4 / 28.0, 11.1 / 15.5, 14.0 / 17.5; output head 168 / 174 and 172 / 182 (1B: equal);
// int4, 5 sequences: QKV 10.8 / 13.0, O 6.8 / 10.4, gate/up 18.0 / 24.4, down 13.2 / 17.7, head 56 / 67; the narrow int4 products
// also from 17 to 32 tokens (steps of up to 6 layers, 17 and 32 sequences: 8B shape 667 / 719 and 736 / 782, 1B shape at 20 and
// 32 380 / 443 and 412 / 468, 8192 columns and 4 layers 906 / 928 and 966 / 988), and their gate/up product where 128 rows a workgroup
// are one round (24 sequences, 8B shape 27.4 / 29.1; a layer of a step, 24 and 32 sequences, 1024 columns 41.3 / 41.8 and 43.2 / 43.2, 2048
// 49.6 / 52.0 and 53.1 / 55.4, 3072 71.3 / 73.2 and 74.8 / 75.9, 4096 84.5 / 86.8 and 89.9 / 91.1, 5120 101.6 / 105.6 and 106.8 / 109.2).  Not the gate/up GEMM
// of the other formats, which has rows for every compute unit without a split (39.0 / 37.6, with FP8 24.6 / 21.9; 1B shape with up
// to 8 tokens 13.4 / 14.6), unless 64 rows per workgroup fill the chip in one round: then up to 8 tokens and, where the other kernel
// has to split k, from 17 on (1B shape, 32 tokens 15.4 / 16.9; a step of 24 sequences with FP8 weights 880 / 896; of 12 and 16
// sequences 904 / 899 and 916 / 911, with FP8 767 / 770 and 776 / 781: within 0.6 %, so those stay).
// FP16 and FP8 weights of other widths: the narrow products by the estimate above against the same for 128 rows a workgroup, with 2.5 us
// for that kernel's shorter pipeline.  Few k splits fit beside many rows and a long k range then reads the activations
// once per 64 rows: 8192 columns, QKV of 640 row groups, 16 and 32 tokens 41.5 / 36.0 and 50.4 / 38.5, with FP8 weights 28.7 / 24.5 and 37.7 /
// 29.5, down projection of 896 k blocks at 32 tokens 86.9 / 81.8 and 59.5 / 51.5; int4 codes cost more to unpack there (down 38.1 / 45.0 at
// 9 tokens).  The output head only where its row tiles are more than one round (32 000 tokens, 4 sequences: 64 k blocks 27.4 / 25.6,
// 160 58.5 / 57.0, with FP8 weights 16 sequences 18.2 / 16.3 and 35.5 / 31.9; 128 256 tokens: above), with FP8 weights also up to 8
// tokens (1B shape 16.7 / 17.4).
// None whose k range leaves half of the wavefronts without a chunk (tiny shape, 4 sequences: 75 us a step, 72 with the other
// kernel; 20 sequences: 80 against 84).
// fp32 sources: two planes double a workgroup's weights, it has two row groups of the residual and wide products and a whole head of
// the QKV product, and its k range is never split.  So only while its rows times k blocks are few (us against skinny_gemm_kernel, models of 4
// layers; residual products, 4 / 12 / 20 / 32 sequences: 16 k blocks 7.9 / 8.7, 8.3 / 8.8, 8.0 / 10.2, 8.4 / 10.4; 32 8.6 / 9.3, 9.7 / 10.0,
// 9.2 / 10.7, 9.9 / 11.1; 64 (1B shape) 11.9 / 11.4, 12.9 / 11.4, 14.3 / 12.8, 15.1 / 13.0; 256 30 / 21, 34 / 21, 38 / 22, 41 / 22.  QKV,
// heads of 64: 32 k blocks 9.9 / 11.1, 11.0 / 11.3, 13.4 / 13.7, 14.2 / 14.2, 48 14.9 / 12.7, 16.5 / 12.6, 19.0 / 14.5, 20.7 / 15.1;
// heads of 128: 16 9.1 / 10.8, 10.2 / 10.8, 12.1 / 13.1, 12.9 / 13.2, 32 13.5 / 11.5, 15.8 / 11.3, 19.1 / 13.6, 21.7 / 14.2.  Wide ones in
// one round, 4 and 12 sequences: gate/up 16 8.7 / 9.0, 9.1 / 9.1, 32 11.5 / 11.8, 12.2 / 11.8; in two rounds 48 21.4 / 18.6, 23.1 / 18.6).
static bool small_gemm_takes(const www_model* m, int epi, int NRG, int KB, int M, const SmallShape& s) {
  if (KB < 16 && M <= 16) return false;
  if (m->wsplit) {
    if (epi == EPI_QKV) return m->hd * KB <= 64 * 32;
    return KB <= 48 && (epi == EPI_RESID || (M <= 8 && NRG <= 2 * decode_wg_target()));
  }
  if (epi == EPI_QKV || epi == EPI_RESID) return m->int4_group || s.us <= general_us(NRG, KB, M, m->fp8 ? 1.f : 2.f) + 2.5f;
  if (M > 16) return epi == EPI_SWIGLU && NRG <= (m->int4_group ? 8 : 4) * decode_wg_target();
  if (m->int4_group) return true;
  if (epi == EPI_LOGITS) return (NRG + 7) / 8 > decode_wg_target() || (m->fp8 && M <= 8);
  return M <= 8 && NRG <= 4 * decode_wg_target();
}

uint64_t small_gemm_partial_bytes(int NRG) { return (uint64_t)NRG * 8 * 2 * 1024; }  // [split][row group][2 token groups]

static SmallShape small_gemm_shape(const www_model* m, int epi, int NRG, int KB, int M) {
  const int xf = M <= 8 ? 1 : M <= 16 ? 2 : 4;
  const bool narrow = epi == EPI_QKV || epi == EPI_RESID;
  if (narrow && !m->wsplit) return narrow_shape(epi, NRG, KB, m->hd, xf, m->int4_group ? WMODE_INT4 : m->fp8 ? WMODE_FP8 : WMODE_F16);
  SmallShape s = {2, 1, xf, 1, (KB + 3) / 4 * 4, 0.f};
  if (m->wsplit) {  // two planes: two row groups fit the registers; whole heads, so that nothing is handed over
    if (epi == EPI_QKV) s.RW = m->hd / 32;
  } else {  // one round of workgroups where the rows allow it
    s.R = 4;
    while (s.RW < (epi == EPI_LOGITS ? 8 : 2) && (NRG + 4 * s.RW - 1) / (4 * s.RW) > decode_wg_target()) s.RW *= 2;
  }
  return s;
}

SmallShape small_gemm_route(const www_model* m, int epi, int NRG, int KB, int M) {
  SmallShape s = {0, 0, 0, 0, 0, 0.f};
  if (M > 32) return s;
  s = small_gemm_shape(m, epi, NRG, KB, M);
  if (!small_gemm_takes(m, epi, NRG, KB, M, s)) s.R = 0;
  return s;
}

// The kernels there are: those that small_gemm_takes and small_gemm_shape lead to (fp16 and FP8 gate/up products take one round of
// workgroups and not 9 to 16 tokens, int4 ones one round from 17 tokens on, output heads of fp16 and FP8 weights more than one round of
// row tiles but for FP8 up to 8 tokens).
static constexpr bool sg_built(int epi, int wmode, int R, int RW, int xf) {
  const bool narrow = epi == EPI_QKV || epi == EPI_RESID;
  if (wmode == WMODE_SPLIT) return R == 2 && (epi == EPI_QKV ? RW == 2 || RW == 4 : RW == 1) && (narrow || xf == 1);
  if (narrow) return RW == 1;
  if (R != 4 || (xf == 4 && epi == EPI_LOGITS)) return false;
  if (epi == EPI_SWIGLU) return wmode == WMODE_INT4 ? RW <= 2 : RW == 1 && xf != 2;
  return wmode == WMODE_INT4 || RW >= 4 || (wmode == WMODE_FP8 && xf == 1);
}
static int sg_wmode(const www_model* m) { return m->wsplit ? WMODE_SPLIT : m->int4_group ? WMODE_INT4 : m->fp8 ? WMODE_FP8 : WMODE_F16; }
bool small_gemm_built(const www_model* m, int epi, const SmallShape& s) { return sg_built(epi, sg_wmode(m), s.R, s.RW, s.xf); }

template <int EPI, int WMODE, int R, int RW, int XF>
static bool launch_small_as(const GemmP& p, hipStream_t st) {
  if constexpr (sg_built(EPI, WMODE, R, RW, XF))
    hipLaunchKernelGGL((small_gemm_kernel<WMODE, EPI, R, RW, XF>), dim3(8 * ((p.row_tiles + 7) / 8) * p.zbs), dim3(64 * SG_NW), 0, st, p);
  return sg_built(EPI, WMODE, R, RW, XF);
}
template <int EPI, int WMODE, int R, int RW>
static bool launch_small_xf(const GemmP& p, int xf, hipStream_t st) {
  return xf == 1 ? launch_small_as<EPI, WMODE, R, RW, 1>(p, st) : xf == 2 ? launch_small_as<EPI, WMODE, R, RW, 2>(p, st) : launch_small_as<EPI, WMODE, R, RW, 4>(p, st);
}
template <int EPI, int WMODE>
static bool launch_small_rows(const GemmP& p, const SmallShape& s, hipStream_t st) {
  if (s.R == 1) return s.RW == 1 && launch_small_xf<EPI, WMODE, 1, 1>(p, s.xf, st);
  if (s.R == 2) return s.RW == 1 ? launch_small_xf<EPI, WMODE, 2, 1>(p, s.xf, st) : s.RW == 2 ? launch_small_xf<EPI, WMODE, 2, 2>(p, s.xf, st) : s.RW == 4 && launch_small_xf<EPI, WMODE, 2, 4>(p, s.xf, st);
  if (s.R != 4) return false;
  return s.RW == 1 ? launch_small_xf<EPI, WMODE, 4, 1>(p, s.xf, st) : s.RW == 2 ? launch_small_xf<EPI, WMODE, 4, 2>(p, s.xf, st)
       : s.RW == 4 ? launch_small_xf<EPI, WMODE, 4, 4>(p, s.xf, st) : s.RW == 8 && launch_small_xf<EPI, WMODE, 4, 8>(p, s.xf, st);
}

template <int EPI>
bool launch_small_gemm(www_model* m, GemmP& p, const SmallShape& s, hipStream_t st) {
  p.ksplit = s.ks;
  p.kb_per_split = s.per;
  p.MT = s.xf == 4 ? 2 : 1;
  p.partial = m->partial;
  p.counters = m->counters;
  p.fault_flag = m->fault_dev;
  p.fence_handover = m->handover_fence;
  if (p.wfactor == 0.f) p.wfactor = 1.f;  // not set: an unscaled matrix
  const int hrg = EPI == EPI_QKV ? p.hd / 16 : s.R * s.RW;
  p.row_tiles = (p.NRG + hrg - 1) / hrg;
  p.zbs = p.ksplit * (EPI == EPI_QKV ? hrg / (s.R * s.RW) : 1);
  switch (sg_wmode(m)) {
    case WMODE_SPLIT: return launch_small_rows<EPI, WMODE_SPLIT>(p, s, st);
    case WMODE_INT4: return launch_small_rows<EPI, WMODE_INT4>(p, s, st);
    case WMODE_FP8: return launch_small_rows<EPI, WMODE_FP8>(p, s, st);
    default: return launch_small_rows<EPI, WMODE_F16>(p, s, st);
  }
}
template bool launch_small_gemm<EPI_QKV>(www_model*, GemmP&, const SmallShape&, hipStream_t);
template bool launch_small_gemm<EPI_RESID>(www_model*, GemmP&, const SmallShape&, hipStream_t);
template bool launch_small_gemm<EPI_SWIGLU>(www_model*, GemmP&, const SmallShape&, hipStream_t);
template bool launch_small_gemm<EPI_LOGITS>(www_model*, GemmP&, const SmallShape&, hipStream_t);
