// Shared by the GEMM kernels: launch arguments and the fused epilogues.
#pragma once
#include "common.h"

struct GemmArgs {
  // what a workgroup needs before it can ask for anything, in one line of the argument buffer
  const uint4* wp;    // weights, fragment order, 64 uint4 per tile (e4m3 codes: per two tiles)
  const uint4* xp;    // activations, fragment order
  const int* n_rows;  // device: rows in use
  uint64_t cut[2];    // one-stream GEMM: how n row tiles (n <= 32) are cut, 4 bits at n - 1 (rows_cut_of)
  int n_rows_val;     // >= 0: the row count is known on the host, n_rows is not read
  int NB;             // weight row blocks (32 output features each)
  int KS;             // K steps (64 k = 4 tiles each)
  int S;              // split-K factor
  int rows_hi;        // the launch has work only if rows_lo <= row count < rows_hi (two kernels share a GEMM)
  int fb_first;       // one-stream GEMM: the feature blocks per workgroup that it assumes until the row count is known
  int rows_lo;
  int x_tiles;        // many-rows GEMM: 32-row tiles the activation buffer holds (copies are clamped to it)
  const float* wscale;  // e4m3 weights: scale per output feature (packed row order), else null
  const uint4* zero_tile;  // 1 KiB of zeros
  float* partial;
  int* counters;
  int* split;         // many-rows GEMM with a residual: where it leaves the split factor it chose
  GemmEpi e;
  NormIn norm;        // fused RMSNorm of the input rows (few-rows kernel only)
};
// e4m3 weights: a lane's 8 codes of one k-tile (two dwords) -> its 8 fp16 operand values.
// The hardware conversion decodes OCP e4m3 (verified code by code); every e4m3 value is an
// fp16 value, so the second conversion is exact.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
template <bool HIGH>
__device__ inline uint32_t e4m3_pair_to_f16(uint32_t codes) {
  const f32x2_t v = __builtin_amdgcn_cvt_pk_f32_fp8((int)codes, HIGH);
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(v.x, v.y));
}
__device__ inline uint4 e4m3_tile_to_f16(uint32_t lo, uint32_t hi) {
  return make_uint4(e4m3_pair_to_f16<false>(lo), e4m3_pair_to_f16<true>(lo),
                    e4m3_pair_to_f16<false>(hi), e4m3_pair_to_f16<true>(hi));
}
// k-tile (2 c + half) of a 16-byte slot that holds the codes of two k-tiles
__device__ inline uint4 e4m3_slot_half(const uint4& slot, int half) {
  return half ? e4m3_tile_to_f16(slot.z, slot.w) : e4m3_tile_to_f16(slot.x, slot.y);
}
// the scales of the 16 results a lane holds of weight block nb (features 8 q + 4 g + i)
__device__ inline void scale_tile(const float* wscale, int nb, int g, f32x16& acc) {
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const float4 s = *(const float4*)(wscale + nb * 32 + 8 * q4 + 4 * g);
    acc[4 * q4] *= s.x; acc[4 * q4 + 1] *= s.y; acc[4 * q4 + 2] *= s.z; acc[4 * q4 + 3] *= s.w;
  }
}

// The arguments that the epilogue needs, read with the first ones
template <int EPI>
__device__ __forceinline__ void read_epilogue_args(const GemmArgs& a) {
  if constexpr (EPI == EPI_QKV)
    read_args(a.e.rows, a.e.rope_cos, a.e.rope_sin, a.e.qbuf, a.e.kv, a.e.kv_stream_stride, a.e.kv_layer_off,
              a.e.n_q_heads, a.e.max_seq);
  else if constexpr (EPI == EPI_RESID) read_args(a.e.rows, a.e.d_model, a.e.rpart, a.e.rpart_rows);
  else if constexpr (EPI == EPI_SWIGLU) read_args(a.e.rows, a.e.xf, a.e.kc_f);
  else read_args(a.e.logits, a.e.logits_stride, a.e.best, a.e.vocab);
}

// x / (1 + e^-x): one step from x times the chip's reciprocal (1 ulp), whose remainder is exact, gives the bits of the
// IEEE division for every fp32 value up to kFarGate (a test runs through all of them; the sign of the remainder is such that a
// negative zero stays one).  Beyond, the reciprocal gets subnormal, which the chip makes 0, and infinities begin.  4
// instructions instead of 11: the division was 1400 of the 3600 that a wave of the many-rows kernel spent on a work item
// of 256 x 256 after its last product.
__device__ inline float silu_quick(float x) {
  const float y = 1.f + __expf(-x), r = __builtin_amdgcn_rcpf(y), q = x * r;
  return fmaf(-fmaf(y, q, -x), r, q);
}
// The same for every value: the reciprocal is taken of a quarter of the denominator and the fix-up treats infinities and NaN as
// the division does.  3 instructions more (gate/up of grouped queries, 32 x 304 tokens, 1 %), and half the code of the division,
// which the one-stream kernel holds once per row tile (decode of 64 streams, d_model 256, 7 tokens: 886 us with that, 861 with this).
__device__ inline float silu_any(float x) {
  const float e = __expf(-x), y = 1.f + e, r = 0.25f * __builtin_amdgcn_rcpf(fmaf(e, 0.25f, 0.25f)), q = x * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-y, q, x), r, q), y, x);
}
// The largest gate of a tile is looked for beside the quick quotients (1 instruction for two gates; asm, because fmaxf makes
// its operands quiet first), and where it is beyond kFarGate the stores are made again with the others.  (A branch
// ahead of every tile's quotients: 3 % of that gate/up.)
constexpr float kFarGate = 87.f;
__device__ __forceinline__ float largest_gate(const f32x16& acc, float most = 0.f) {
#pragma unroll
  for (int k = 0; k < 8; k += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(acc[k]), "v"(acc[k + 1]));
  return most;
}

// What an epilogue reads from memory for one tile: rotary factors of a query or key block, residual rows of a
// projection.  It is asked for apart from what is done with it: behind the stores of another tile the compiler
// keeps a load where it is (they might overlap), and every tile would be a round trip of its own.
template <int EPI>
struct EpiIn {};
template <>
struct EpiIn<EPI_QKV> { float4 c[2], s[2]; };
template <>
struct EpiIn<EPI_RESID> { float4 r[4]; };

template <int EPI>
__device__ __forceinline__ void epilogue_load(const GemmEpi& e, int nb, int id, int g, EpiIn<EPI>& in) {
  if constexpr (EPI == EPI_QKV) {
    const int half = e.head_dim >> 1, bph = e.head_dim >> 5;  // (2 or 4 blocks per head)
    if (nb < (e.n_q_heads + e.n_kv_heads) * bph) {
      const size_t at = (size_t)(id & 0xffff) * half + 16 * (nb & (bph - 1)) + 4 * g;
#pragma unroll
      for (int q4 = 0; q4 < 2; ++q4) {
        in.c[q4] = *(const float4*)(e.rope_cos + at + 8 * q4);
        in.s[q4] = *(const float4*)(e.rope_sin + at + 8 * q4);
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
    const float* rs = e.resid_src + ((size_t)(id >> 16) * e.resid_seq_stride + (e.h_compact ? 0 : id & 0xffff)) * e.d_model +
                      nb * 32 + 4 * g;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) in.r[q4] = *(const float4*)(rs + 8 * q4);
  }
}

// FAR (SwiGLU): for gates beyond kFarGate
template <int EPI, bool F16, bool FAR = false>
__device__ __forceinline__ void epilogue_store(const GemmEpi& e, int nb, int slot, int id, int g,
                                               const f32x16& acc, const EpiIn<EPI>& in) {
  const int b = id >> 16, pos = id & 0xffff;
  if constexpr (EPI == EPI_QKV) {
    const int hd = e.head_dim, bph = hd >> 5, bph_log = (hd >> 7) + 1;  // (hd is 64 or 128)
    const int nbq = e.n_q_heads * bph, nbk = e.n_kv_heads * bph;
    const size_t head_elems = (size_t)e.max_seq * hd;
    bf16_t* kvl = e.kv + (size_t)b * e.kv_stream_stride + e.kv_layer_off;
    if (nb < nbq + nbk) {
      // query or key block: rows 0..15 hold features f, rows 16..31 their rotary partners f + hd/2
      const bool isq = nb < nbq;
      const int nbl = isq ? nb : nb - nbq, head = nbl >> bph_log, sb = nbl & (bph - 1);
      bf16_t* dst;
      int row;  // row of the fragment-ordered destination
      if (isq) {
        dst = e.qbuf + ((size_t)(slot >> 5) * e.n_q_heads + head) * (size_t)(hd >> 4) * 512;
        row = slot & 31;
      } else {
        dst = kvl + (size_t)head * head_elems + (size_t)(pos >> 5) * (hd >> 4) * 512;
        row = pos & 31;
      }
#pragma unroll
      for (int q4 = 0; q4 < 2; ++q4) {
        const int f1 = 16 * sb + 8 * q4 + 4 * g;
        const float4 c4 = in.c[q4], s4 = in.s[q4];
        const float cs[4] = {c4.x, c4.y, c4.z, c4.w}, sn[4] = {s4.x, s4.y, s4.z, s4.w};
        float o1[4], o2[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float x1 = acc[4 * q4 + k], x2 = acc[4 * (q4 + 2) + k];
          // (which product is rounded is written out: left to the compiler it changes with the code around it,
          // and with it the last bits of every result)
          o1[k] = fmaf(x1, cs[k], -(x2 * sn[k]));
          o2[k] = fmaf(x2, cs[k], x1 * sn[k]);
        }
        const int f2 = f1 + (hd >> 1);
        *(uint2*)(dst + (size_t)(f1 >> 4) * 512 + ((row + (((f1 >> 3) & 1) << 5)) << 3) + (f1 & 7)) =
            make_uint2(pack_op2<F16>(o1[0], o1[1]), pack_op2<F16>(o1[2], o1[3]));
        *(uint2*)(dst + (size_t)(f2 >> 4) * 512 + ((row + (((f2 >> 3) & 1) << 5)) << 3) + (f2 & 7)) =
            make_uint2(pack_op2<F16>(o2[0], o2[1]), pack_op2<F16>(o2[2], o2[3]));
      }
    } else {
      // value block -> the cache's V tile: per 32 positions and 32 features, the
      // operand of the P.V product (key order inside a tile follows the score tile)
      const int nbl = nb - nbq - nbk, head = nbl >> bph_log, ib = nbl & (bph - 1);
      const int pt = pos >> 5, pl = pos & 31, s = pl >> 4, r16 = pl & 15;
      const int gp = (r16 & 7) >> 2, ep = 4 * (r16 >> 3) + (r16 & 3);
      bf16_t* dst = kvl + (size_t)(e.n_kv_heads + head) * head_elems +
                    (((size_t)pt * bph + ib) * 2 + s) * 512 + (size_t)(32 * gp) * 8 + ep;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
          const uint32_t two = pack_op2<F16>(acc[4 * q4 + k], acc[4 * q4 + k + 1]);
          dst[(8 * q4 + 4 * g + k) * 8] = (bf16_t)two;
          dst[(8 * q4 + 4 * g + k + 1) * 8] = (bf16_t)(two >> 16);
        }
    }
  } else if constexpr (EPI == EPI_RESID) {
    const int hpos = e.h_compact ? 0 : pos;
    float* hp = e.h + ((size_t)b * e.h_seq_stride + hpos) * e.d_model + nb * 32 + 4 * g;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      float4 r = in.r[q4];
      r.x += acc[4 * q4]; r.y += acc[4 * q4 + 1]; r.z += acc[4 * q4 + 2]; r.w += acc[4 * q4 + 3];
      *(float4*)(hp + 8 * q4) = r;
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // rows 0..15 of the block: gate features, rows 16..31: the matching up features
#pragma unroll
    for (int q4 = 0; q4 < 2; ++q4) {
      const int ff = 16 * nb + 8 * q4 + 4 * g;
      float o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = acc[4 * q4 + k];
        o[k] = (FAR ? silu_any(x) : silu_quick(x)) * acc[4 * (q4 + 2) + k];
      }
      *(uint2*)(e.xf + frag_off(slot, ff, e.kc_f)) =
          make_uint2(pack_op2<F16>(o[0], o[1]), pack_op2<F16>(o[2], o[3]));
    }
  } else {  // EPI_LOGITS: slot is the stream
    // (with the logits the greatest of the block's 32 and its token, ties -> lower id, a NaN never: what is
    // left for the argmax are vocab / 32 pairs)
    float v = -INFINITY;
    int token = 0x7fffffff;
    auto take = [&](float x, int t) {
      if (x > v || (x == v && t < token)) { v = x; token = t; }
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) take(acc[i], nb * 32 + 8 * (i >> 2) + 4 * g + (i & 3));
    const float v2 = __shfl_xor(v, 32);
    take(v2, __shfl_xor(token, 32));
    if (g == 0) e.best[(size_t)slot * (e.vocab >> 5) + nb] = make_float2(v, __int_as_float(token));
    float* out = e.logits + (size_t)slot * e.logits_stride + nb * 32 + 4 * g;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *(float4*)(out + 8 * q4) =
          make_float4(acc[4 * q4], acc[4 * q4 + 1], acc[4 * q4 + 2], acc[4 * q4 + 3]);
  }
}

template <int EPI, bool F16>
__device__ __forceinline__ void epilogue_tile(const GemmEpi& e, int nb, int slot, int id, int g, const f32x16& acc) {
  EpiIn<EPI> in;
  epilogue_load<EPI>(e, nb, id, g, in);
  epilogue_store<EPI, F16>(e, nb, slot, id, g, acc, in);
  if constexpr (EPI == EPI_SWIGLU)
    if (__builtin_expect(__any(largest_gate(acc) > kFarGate), 0)) epilogue_store<EPI, F16, true>(e, nb, slot, id, g, acc, in);
}

// gemm_tall.hip: the many-rows kernel with both operands through LDS (its plan: common.h).
// The caller has filled every field of `a` except S and x_tiles; S_max: most K splits
// (1 unless the projection adds to the residual stream).
void launch_gemm_tall(bool f16, int epi, GemmArgs& a, int rows_cap, int S_max, hipStream_t st);
int gemm_tall_init();  // kernel attribute setup; returns hipError_t
// e4m3 weight codes (n_slots slots of two k-tiles, 64 uint4 each) -> fp16 tiles, fragment order
void launch_expand_e4m3(const uint4* codes, uint4* tiles, size_t n_slots, hipStream_t st);
