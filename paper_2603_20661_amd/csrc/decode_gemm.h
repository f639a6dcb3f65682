// Shared by the kernels of the decode path: parameters of its GEMMs, layout of the packed activations, unpacking of the
// weight-only formats.
#pragma once
#include "common.h"

#define NEG_INF (-__builtin_inff())

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// offset (in elements) of column k of token t in a packed activation buffer with MT token groups
__device__ __forceinline__ int64_t packed_x_offset(int k, int t, int MT, int hl) {
  int kb = k >> 5, g = (k & 31) >> 3, e = k & 7;
  return ((((int64_t)kb * MT + (t >> 4)) * 2 + hl) * 64 + g * 16 + (t & 15)) * 8 + e;
}

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

struct GemmP {
  const u32x4* W;    // packed weights, 16-byte units (fp16 fragments, or FP8 codes of two k blocks)
  const u32x4* Wlo;  // low-order plane (fp32 sources) or null
  float wfactor;     // FP8 weights: the matrix's scale, applied to the result
  const u32x2* Wscale;  // int4 weights: four fp16 group scales per (chunk of 4 k blocks, row)
  int NRG, KB;       // row groups of 16, k blocks of 32
  const u32x4* X;    // packed activations
  int MT, M;         // token groups in X, valid tokens
  int kb_per_split, ksplit;
  int row_tiles, zbs;  // grid: 8 * ceil(row_tiles / 8) * ksplit * zbs workgroups; small_gemm_kernel: hand-over groups, workgroups of one
  int fence_handover;  // 1: workgroups of one row tile may sit behind different L2s
  float* partial;    // [ksplit][zbs][row_tiles] tiles of 128 rows x 16 MTK tokens
  unsigned long long* counters;  // [zbs][row_tiles]: arrivals in bits 0-7, arrivals per XCD in eight 5-bit fields above
  int* fault_flag;   // host-visible; set when the splits of a row tile turn out to sit on different XCDs
  const float* ssq_in;  // [token][SSQ_TILES], up to 32 tokens [token][SSQ_ROWS]; row scale = rsqrt(sum of the first n_ssq_in entries / dim + eps); null: no scale
  int n_ssq_in;
  float inv_dim, eps;
  // QKV epilogue
  uint16_t *q_hi, *q_lo;
  float qscale;
  uint16_t *kplane, *vplane;  // this layer's K and V planes of the pool (16-bit codes)
  float* kvscale;             // and its plane of scales
  const int32_t *seq_lens, *table;
  int mbs, hd, Hq, Hkv;
  const float2* rope;
  const float* qk_gain;  // models with normalised query / key heads: [2][hd] gains in packed row order; null otherwise
  // residual epilogue
  float* h;
  const float* gain_next;
  uint16_t* xnext;
  float* ssq_out;
  int d;
  // SwiGLU epilogue
  uint16_t* xa;
  int F;
  // logits epilogue
  float* logits;
  int V;
  float* best_val;  // [token][workgroups over the rows] largest logit of a workgroup's rows and its index; null: nobody asks for the tokens
  int* best_idx;
};

// the larger of two logits, the lowest index winning ties (a NaN is never taken)
__device__ __forceinline__ void argmax_take(float& best, int& bi, float v, int i) {
  if (v > best || (v == best && i < bi)) { best = v; bi = i; }
}
// ... of a token over the four lanes l, l ^ 16, l ^ 32 and l ^ 48
__device__ __forceinline__ void argmax_of_rows(float& best, int& bi) {
  argmax_take(best, bi, __shfl_xor(best, 16), __shfl_xor(bi, 16));
  argmax_take(best, bi, __shfl_xor(best, 32), __shfl_xor(bi, 32));
}

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// 8 FP8 E4M3 codes (two 32-bit words, lowest byte first) -> 8 fp16 values, exact (|value| <= 448); the conversion
// instruction widens two codes at a time.
__device__ __forceinline__ f16x8 fp8x8_to_f16x8(uint32_t lo, uint32_t hi) {
  const f16x2 a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, false), b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, true);
  const f16x2 c = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, false), d = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, true);
  return __builtin_shufflevector(__builtin_shufflevector(a, b, 0, 1, 2, 3), __builtin_shufflevector(c, d, 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// 8 four-bit codes (one 32-bit word, the codes of columns 2 i and 2 i + 1 in nibbles i and i + 4: one per half) -> 8 fp16 values
// (code - 8) * scale.  A code n is planted in the mantissa of the fp16 numbers 1024 (0x6400 | n = 1024 + n) or 64 (0x5400 | n << 4 = 64 + n),
// both exact; 1032 or 72 is subtracted and the result multiplied by the group's scale, two values per instruction; with a scale of 8
// significant bits (bf16) the product is exact.  13 instructions for 8 weights; with the codes in column order 19, two nibbles of a pair
// being brought together by a byte permutation.
__device__ __forceinline__ f16x8 int4x8_to_f16x8(uint32_t w, f16x2 scale) {
  const f16x2 off[2] = {{(_Float16)1032.f, (_Float16)1032.f}, {(_Float16)72.f, (_Float16)72.f}};
  f16x2 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t pair;  // one instruction: of (w & mask) | bits with two literals the compiler makes two
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(pair) : "v"(w), "s"(i & 1 ? 0x00F000F0u : 0x000F000Fu), "v"(i & 1 ? 0x54005400u : 0x64006400u));
    v[i] = (__builtin_bit_cast(f16x2, pair) - off[i & 1]) * scale;
    if (i == 1) w >>= 8;
  }
  return __builtin_shufflevector(__builtin_shufflevector(v[0], v[1], 0, 1, 2, 3), __builtin_shufflevector(v[2], v[3], 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
}

// WMODE: 0 = fp16 weights; 1 = fp16 hi + lo planes (fp32 sources); 2 = FP8 codes, two k blocks per 16-byte unit, widened
// to fp16 in registers just before the MFMAs (the matrix's scale multiplies the result in the epilogue); 3 = int4 codes,
// four k blocks (one chunk) per 16-byte unit, widened and multiplied by their group's scale in registers
enum { WMODE_F16 = 0, WMODE_SPLIT = 1, WMODE_FP8 = 2, WMODE_INT4 = 3 };

// decode_small.hip: GEMMs of a step of up to 32 tokens
int decode_wg_target();  // compute units (decode.hip)
void choose_split(int row_tiles, int zb, int KB, int* ksplit, int* kb_per_split);  // k splits of skinny_gemm_kernel
// 16 R RW rows a workgroup, XF, k splits, k blocks of one; narrow ones: estimate.  R = 0: the GEMM runs in skinny_gemm_kernel
struct SmallShape { int R, RW, xf, ks, per; float us; };
SmallShape small_gemm_route(const www_model* m, int epi, int NRG, int KB, int M);
bool small_gemm_built(const www_model* m, int epi, const SmallShape& s);
template <int EPI>
bool launch_small_gemm(www_model* m, GemmP& p, const SmallShape& s, hipStream_t st);  // false: the shape has no kernel, nothing was launched

// decode_mid.hip: residual GEMMs of a step of 33 to 64 tokens; 16 R rows a workgroup, k splits, k blocks of one.  R = 0: skinny_gemm_kernel
struct MidShape { int R, ks, per; };
MidShape mid_gemm_route(const www_model* m, int epi, int NRG, int KB, int M);
bool mid_gemm_built(const www_model* m, const MidShape& s);
bool launch_mid_gemm(www_model* m, GemmP& p, const MidShape& s, hipStream_t st);  // false: the shape has no kernel, nothing was launched
