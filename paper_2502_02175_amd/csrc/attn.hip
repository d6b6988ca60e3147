// Causal attention of the recomputed queries over the mixed KV cache, and the
// text-to-vision attention statistic (VLA-Cache appendix "Token Reuse
// Mechanism": newly computed tokens update their cache entries, reused tokens
// keep last step's, and attention over that partially updated cache is valid;
// Sec. 3.3, Eq. avistext for the statistic; Sec. 3.1 for the attention itself).
//
// A workgroup handles 32 query rows of one head; its 4 waves take every 4th tile
// of 32 cache positions, flash-style, entirely on the matrix cores,
// and merge their (max, sum, output) triples through LDS at the end:
//   S^T[key, query] = K . Q^T   A operand: K tile (fragment order in the cache),
//                               B operand: Q tile (fragment order from the QKV epilogue)
//   O^T[feat, query] += V^T . P^T  A operand: V tile (the cache stores V per 32
//                               positions already transposed and in the key order
//                               in which a lane holds its scores), B operand: P
// so a lane owns one query column throughout: the running max / sum are
// per-lane scalars (one exchange between the two half-waves per tile) and P goes
// from the score registers straight into the next MFMA.
// Rows are the recomputed rows of the layer, sorted by position inside each
// stream; a query at position p sees cache positions 0..p, fresh or reused.
//
// Statistic: waves whose tile holds text queries run a second pass over the
// vision keys with the final max/sum, sum the probabilities over their text
// rows, and park the sums; the last workgroup of a stream to arrive (atomic
// counter, no waiting) adds the parked sums over heads and tiles in fixed order.
#include "common.h"

struct AttnArgs {
  const int* rows;      // this layer's rows (b << 16 | pos)
  const int* slot_off;  // [B + 1] first slot of every stream
  int decode_pos;       // attn_decode_kernel: one row per stream at this position; rows / slot_off are not read
  const bf16_t* qbuf;
  bf16_t* out;          // attention output, fragment order, KC = kc_out
  int kc_out;
  const bf16_t* kv;     // cache base (stream 0) of this layer
  size_t kv_stream_stride;
  int n_q_heads, n_kv_heads, max_seq;
  int L_v, L_t;
  float scale_log2e;    // log2(e) / sqrt(head_dim)
  float* attn_mean;     // [B, L_v] of this layer or NULL
  int attn_mean_stride; // elements between streams
  float* statp;         // [B][Hq][TT][lv_pad] (of this layer, if the reduction is deferred)
  int TT, lv_pad;
  int* stat_counters;   // [B]
  int defer_stats;      // the parked sums are added up by stats_reduce_kernel after the last layer
  int rows4_from;       // > 0: streams with at least this many rows are left to attn_rows4_kernel
};

// Two probabilities -> one operand dword.  They lie in [0, 256], so the fp16 conversion
// (round to nearest even, as everywhere) needs no saturation.
template <bool F16>
__device__ inline uint32_t pack_p2(float lo, float hi) {
  if constexpr (F16) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
  } else {
    return pack_op2<false>(lo, hi);
  }
}

// Two workgroups per CU: the next tile's K lands in the registers of this one's, and the waves merge one
// feature block each instead of one wave all of them, so that a wave keeps within 256 registers without
// spills (364 before, one workgroup per CU: 288 workgroups of 9 query tiles x 32 heads took two rounds).
// 7B, one stream: 288 rows 19.1 -> 14.6 us, 519 of 601 rows 34.4 -> 26.0, bf16 42.2 -> 28.5, 109 rows 12.6 -> 11.
template <int HD, bool F16>
__global__ __launch_bounds__(256, 2) void attn_rows_kernel(AttnArgs a) {
  constexpr int NC = HD / 16;  // k-tiles of a head
  constexpr int NI = HD / 32;  // feature blocks of a head
  __shared__ float cmb[4][2 + (HD == 128 ? 3 : 2) * 16][64];  // the waves park (max, sum, the blocks they do not finish) here
  __shared__ float fin[2][64];               // merged max and 1/sum per lane
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31, g = lane >> 5;
  const int b = blockIdx.z;
  read_args(a.rows, a.qbuf, a.out, a.kc_out, a.kv, a.kv_stream_stride, a.n_q_heads, a.n_kv_heads, a.max_seq, a.L_v, a.L_t,
            a.scale_log2e, a.attn_mean, a.statp, a.TT, a.lv_pad, a.defer_stats, a.rows4_from);
  const int off_b = ld_scalar(a.slot_off + b);
  const int n_b = ld_scalar(a.slot_off + b + 1) - off_b;
  // The heads are the fastest index: workgroup id % 8, the XCD, is then the same for all query tiles of a head
  // (8 heads or a multiple of them), which share its K and V in that L2; the last tile, whose walk over the cache is
  // the longest, starts first.  (Tiles fastest, every L2 fetched the whole cache, and a last round of workgroups
  // held long walks: 519 of 601 rows of 7B, bf16, 24.2 us, now 19.7; one round of workgroups, 288 rows, 14.5 and 14.5.)
  const int n_qt = (n_b + 31) >> 5, qt = n_qt - 1 - (int)blockIdx.y;
  if (qt < 0) return;
  if (a.rows4_from > 0 && n_b >= a.rows4_from) return;
  const int s0 = qt * 32;
  const int h = blockIdx.x, hk = h / (a.n_q_heads / a.n_kv_heads);
  const bool valid = s0 + j < n_b;
  const int sg = off_b + (valid ? s0 + j : n_b - 1);  // this lane's query slot
  const int pos = valid ? (a.rows[sg] & 0xffff) : 0;
  const int pos_last = ld_scalar(a.rows + off_b + min(s0 + 31, n_b - 1)) & 0xffff;
  const int n_kt = (pos_last >> 5) + 1;

  const size_t head_elems = (size_t)a.max_seq * HD;
  const bf16_t* kbase = a.kv + (size_t)b * a.kv_stream_stride + (size_t)hk * head_elems +
                        (size_t)lane * 8;
  const bf16_t* vbase = kbase + (size_t)a.n_kv_heads * head_elems;

  uint4 qf[NC];
  {
    const bf16_t* qsrc = a.qbuf + ((size_t)(sg >> 5) * a.n_q_heads + h) * (size_t)NC * 512 +
                         (size_t)(((sg & 31) + 32 * g) << 3);
#pragma unroll
    for (int c = 0; c < NC; ++c) qf[c] = *(const uint4*)(qsrc + (size_t)c * 512);
  }
  auto load_k = [&](int kt, uint4(&kf)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *(const uint4*)(kbase + ((size_t)kt * NC + c) * 512);
  };
  auto scores = [&](const uint4(&kf)[NC], f32x16& s) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) s = mfma32<F16>(kf[c], qf[c], s);
  };

  f32x16 o[NI];
#pragma unroll
  for (int ib = 0; ib < NI; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[ib][i] = 0.f;
  float m = -INFINITY, l = 0.f;

  uint4 kf[NC];
  if (w < n_kt) load_k(w, kf);
  for (int kt = w; kt < n_kt; kt += 4) {
    f32x16 s;
    scores(kf, s);
    __builtin_amdgcn_sched_barrier(0);
    uint4 vf[NI * 2];  // this tile's V, and the next tile's K in the registers of this one's, fly during the softmax
#pragma unroll
    for (int t = 0; t < NI * 2; ++t) vf[t] = *(const uint4*)(vbase + ((size_t)kt * NI * 2 + t) * 512);
    if (kt + 4 < n_kt) load_k(kt + 4, kf);
    __builtin_amdgcn_sched_barrier(0);
    // register 4*q4 + e of a lane is key 32*kt + 8*q4 + 4*g + e
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kp = 32 * kt + 8 * (i >> 2) + 4 * g + (i & 3);
      s[i] = (kp <= pos) ? s[i] * a.scale_log2e : -INFINITY;
      tmax = fmaxf(tmax, s[i]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    // a tile that lies wholly behind this query leaves max at -inf: keep the state as it is
    const float m_new = fmaxf(m, tmax);
    const float alpha = (m_new == -INFINITY) ? 1.f : exp2f(m - m_new);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    m = m_new;
    float psum = 0.f;
    float pr[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      pr[i] = exp2f(s[i] - m_use);
      psum += pr[i];
    }
    l = l * alpha + psum;
    uint4 pb[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      pb[t].x = pack_p2<F16>(pr[8 * t + 0], pr[8 * t + 1]);
      pb[t].y = pack_p2<F16>(pr[8 * t + 2], pr[8 * t + 3]);
      pb[t].z = pack_p2<F16>(pr[8 * t + 4], pr[8 * t + 5]);
      pb[t].w = pack_p2<F16>(pr[8 * t + 6], pr[8 * t + 7]);
    }
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[ib][i] *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t) o[ib] = mfma32<F16>(vf[ib * 2 + t], pb[t], o[ib]);
    }
  }
  l += __shfl_xor(l, 32);

  // Merge the 4 waves, wave ib the feature block ib of all of them, in the order of the waves (wave 0
  // owns tile 0, so its max is finite: key 0 is visible to every query)
  f32x16 own;
  cmb[w][0][lane] = m;
  cmb[w][1][lane] = l;
#pragma unroll
  for (int ib = 0; ib < NI; ++ib) {
    if (ib == w) own = o[ib];
    else {
#pragma unroll
      for (int i = 0; i < 16; ++i) cmb[w][2 + (w < ib ? ib - 1 : ib) * 16 + i][lane] = o[ib][i];
    }
  }
  __syncthreads();
  if (w < NI) {
    f32x16 acc;
    m = cmb[0][0][lane];
    l = cmb[0][1][lane];
    // (as a loop it moved the 16 sums of every turn: 80 rows of the tiny shape 155.4 -> 154.2 us)
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
      f32x16 t = own;
      if (ww != w) {
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = cmb[ww][2 + (ww < w ? w - 1 : w) * 16 + i][lane];
      }
      if (ww == 0) {
        acc = t;
        continue;
      }
      const float m_w = cmb[ww][0][lane], l_w = cmb[ww][1][lane];
      const float m_new = fmaxf(m, m_w);
      const float a0 = exp2f(m - m_new), a1 = exp2f(m_w - m_new);
      m = m_new;
      l = fmaf(l, a0, l_w * a1);
      // (which of the two products is rounded is written out: left to the compiler it changed with the
      // code around it, and with it the last bits of every result)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = fmaf(acc[i], a0, t[i] * a1);
    }
    const float inv = 1.f / l;
    if (w == 0) {
      fin[0][lane] = m;
      fin[1][lane] = (valid && pos >= a.L_v) ? inv : 0.f;  // (the statistic counts text rows only)
    }
    if (valid) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int f = h * HD + 32 * w + 8 * q4 + 4 * g;
        *(uint2*)(a.out + frag_off(sg, f, a.kc_out)) =
            make_uint2(pack_op2<F16>(acc[4 * q4] * inv, acc[4 * q4 + 1] * inv),
                       pack_op2<F16>(acc[4 * q4 + 2] * inv, acc[4 * q4 + 3] * inv));
      }
    }
  }

  // ---- text-to-vision statistic (all conditions are uniform over the workgroup) ----
  if (!a.attn_mean || a.L_t <= 0 || a.L_v <= 0) return;
  if (pos_last < a.L_v) return;  // no text row in this tile
  __syncthreads();
  const int x_first = (n_b - a.L_t) >> 5;  // first tile that holds a text row
  const int n_tt = ((n_b - 1) >> 5) - x_first + 1;
  const int tt = qt - x_first;
  float* park = a.statp + (((size_t)b * a.n_q_heads + h) * a.TT + tt) * a.lv_pad;
  const int n_vt = (a.L_v + 31) >> 5;
  // Here the scores are taken the other way round, Q K^T: a lane's column is a KEY and its 16
  // registers are queries (8 q4 + 4 g + e, whose reference point and 1/sum wave 0 left in
  // LDS), so the sum over the queries of the tile is 16 additions in the lane and one
  // exchange between the two halves of the wave.
  const float* m_q = fin[0] + 4 * g;
  const float* inv_q = fin[1] + 4 * g;
  if (w < n_vt) load_k(w, kf);
  for (int kt = w; kt < n_vt; kt += 4) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) s = mfma32<F16>(qf[c], kf[c], s);
    if (kt + 4 < n_vt) load_k(kt + 4, kf);  // the next tile flies during the arithmetic
    float r = 0.f;  // fixed order: the lane's 16 queries, then the other half's
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int qi = 8 * (i >> 2) + (i & 3);
      const float iq = inv_q[qi];
      r += iq != 0.f ? exp2f(s[i] * a.scale_log2e - m_q[qi]) * iq : 0.f;
    }
    r += __shfl_xor(r, 32);
    if (g == 0) {
      if (a.defer_stats) park[32 * kt + j] = r;  // read by a later kernel: plain stores
      else st_coherent(park + 32 * kt + j, r);
    }
  }
  if (a.defer_stats) return;
  stores_done();
  __syncthreads();
  if (tid == 0) {
    const int expect = a.n_q_heads * n_tt;
    const int old = atomicAdd(a.stat_counters + b, 1);
    s_last = (old == expect - 1);
    if (old == expect - 1) a.stat_counters[b] = 0;
  }
  __syncthreads();
  if (!s_last) return;
  // the parked sums of all heads and text tiles, in fixed order, 16 loads in flight at a time
  const float norm = 1.f / ((float)a.n_q_heads * (float)a.L_t);
  const int n_part = a.n_q_heads * n_tt;
  const float* part0 = a.statp + (size_t)b * a.n_q_heads * a.TT * a.lv_pad;
  for (int v = tid; v < a.L_v; v += 256) {
    float acc = 0.f;
    for (int p0 = 0; p0 < n_part; p0 += 16) {
      float t[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int p = min(p0 + i, n_part - 1), hh = p / n_tt, tq = p - hh * n_tt;
        t[i] = ld_coherent(part0 + ((size_t)hh * a.TT + tq) * a.lv_pad + v);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) acc += (p0 + i < n_part) ? t[i] : 0.f;
    }
    a.attn_mean[(size_t)b * a.attn_mean_stride + v] = acc * norm;
  }
}

// ---------------------------------------------------------------------------
// One query per stream and head (a decode pass).  The query heads that share a kv head fill the
// columns of one tile (at most 32 of them), so a workgroup per stream and kv head reads K and V
// once for all of them.  Bound by latency: a stream's cache slice of a layer is a few MB, read by
// as many workgroups as there are kv heads.  So every wave takes key tiles of its own (one each up
// to 16 tiles, 512 positions), asks for its query, K and V at once, and the waves meet once, in
// LDS, where only the columns that hold a query are exchanged.  (MULTI: more tiles than that; 8
// waves, whose query stays in registers beside the next tile.)  7B shape, one stream, 294
// positions: 6.1 us per launch against 8.7 with 4 waves that walked three tiles each and
// exchanged whole tiles; grouped queries, 32 streams, 310 positions: 6.7 against 9.0.
// ---------------------------------------------------------------------------
constexpr int kDecWaves = 16, kDecWavesMulti = 8;  // 4 and 2 per SIMD: 128 and 256 registers a wave

template <int HD, bool F16, bool MULTI>
__global__ __launch_bounds__(64 * (MULTI ? kDecWavesMulti : kDecWaves)) void attn_decode_kernel(AttnArgs a) {
  constexpr int NC = HD / 16;  // k-tiles of a head
  constexpr int NI = HD / 32;  // feature blocks of a head
  extern __shared__ float dec_lds[];  // [waves][columns][HD + 4]: output, reference point, sum
  read_args(a.decode_pos, a.qbuf, a.out, a.kc_out, a.kv, a.kv_stream_stride, a.n_q_heads, a.n_kv_heads, a.max_seq, a.scale_log2e);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int j = lane & 31, g = lane >> 5;
  const int b = blockIdx.y, group = a.n_q_heads / a.n_kv_heads, per_kv = (group + 31) >> 5;
  const int hk = blockIdx.x / per_kv, c0 = (blockIdx.x - hk * per_kv) * 32;
  const int nc = min(group - c0, 32);           // columns that hold a query
  const int h0 = hk * group + c0, h = h0 + min(j, nc - 1);
  const int pos = a.decode_pos, n_kt = (pos >> 5) + 1;

  const size_t head_elems = (size_t)a.max_seq * HD;
  const bf16_t* kbase = a.kv + (size_t)b * a.kv_stream_stride + (size_t)hk * head_elems + (size_t)lane * 8;
  const bf16_t* vbase = kbase + (size_t)a.n_kv_heads * head_elems;
  uint4 qf[NC], kf[NC], vf[NI * 2];
  const bf16_t* qsrc = a.qbuf + ((size_t)(b >> 5) * a.n_q_heads + h) * (size_t)NC * 512 + (size_t)(((b & 31) + 32 * g) << 3);
#pragma unroll
  for (int c = 0; c < NC; ++c) qf[c] = *(const uint4*)(qsrc + (size_t)c * 512);
  auto load_k = [&](int kt) {
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *(const uint4*)(kbase + ((size_t)kt * NC + c) * 512);
  };
  auto load_v = [&](int kt) {
#pragma unroll
    for (int t = 0; t < NI * 2; ++t) vf[t] = *(const uint4*)(vbase + ((size_t)kt * NI * 2 + t) * 512);
  };
  load_k(min(w, n_kt - 1));
  load_v(min(w, n_kt - 1));
  __builtin_amdgcn_sched_barrier(0);

  f32x16 o[NI];
#pragma unroll
  for (int ib = 0; ib < NI; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[ib][i] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int kt = w; kt < n_kt; kt += nw) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) s = mfma32<F16>(kf[c], qf[c], s);
    if (MULTI && kt + nw < n_kt) load_k(kt + nw);  // (flies during softmax and P.V)
    // register 4*q4 + e of a lane is key 32*kt + 8*q4 + 4*g + e
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kp = 32 * kt + 8 * (i >> 2) + 4 * g + (i & 3);
      s[i] = (kp <= pos) ? s[i] * a.scale_log2e : -INFINITY;
      tmax = fmaxf(tmax, s[i]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    const float m_new = fmaxf(m, tmax);  // (a tile holds at least one visible key)
    const float alpha = (m_new == -INFINITY) ? 1.f : exp2f(m - m_new);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    m = m_new;
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = exp2f(s[i] - m_use);
      psum += s[i];
    }
    l = l * alpha + psum;
    uint4 pb[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      pb[t].x = pack_p2<F16>(s[8 * t + 0], s[8 * t + 1]);
      pb[t].y = pack_p2<F16>(s[8 * t + 2], s[8 * t + 3]);
      pb[t].z = pack_p2<F16>(s[8 * t + 4], s[8 * t + 5]);
      pb[t].w = pack_p2<F16>(s[8 * t + 6], s[8 * t + 7]);
    }
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[ib][i] *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t) o[ib] = mfma32<F16>(vf[ib * 2 + t], pb[t], o[ib]);
    }
    if (!MULTI) break;
    if (kt + nw < n_kt) load_v(kt + nw);
  }
  l += __shfl_xor(l, 32);

  constexpr int ROW = HD + 4;
  if (j < nc) {
    float* mine = dec_lds + ((size_t)w * nc + j) * ROW;
#pragma unroll
    for (int ib = 0; ib < NI; ++ib)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(float4*)(mine + 32 * ib + 8 * q4 + 4 * g) =
            make_float4(o[ib][4 * q4], o[ib][4 * q4 + 1], o[ib][4 * q4 + 2], o[ib][4 * q4 + 3]);
    if (g == 0) {
      mine[HD] = m;
      mine[HD + 1] = l;
    }
  }
  __syncthreads();
  // 4 features of one column per thread; the waves' parts in order (wave 0 has tile 0, whose
  // first key every query sees, so M is finite)
  const int n_w = min(nw, n_kt);
  for (int e = tid; e < nc * (HD / 4); e += blockDim.x) {
    const int col = e / (HD / 4), f = (e - col * (HD / 4)) * 4;
    const float* src = dec_lds + (size_t)col * ROW;
    const size_t step = (size_t)nc * ROW;
    float M = src[HD];
    for (int ww = 1; ww < n_w; ++ww) M = fmaxf(M, src[ww * step + HD]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float L = 0.f;
    for (int ww = 0; ww < n_w; ++ww) {
      const float sc = exp2f(src[ww * step + HD] - M);
      const float4 x = *(const float4*)(src + ww * step + f);
      acc.x += sc * x.x; acc.y += sc * x.y; acc.z += sc * x.z; acc.w += sc * x.w;
      L += sc * src[ww * step + HD + 1];
    }
    const float inv = 1.f / L;
    *(uint2*)(a.out + frag_off(b, (h0 + col) * HD + f, a.kc_out)) =
        make_uint2(pack_op2<F16>(acc.x * inv, acc.y * inv), pack_op2<F16>(acc.z * inv, acc.w * inv));
  }
}

// ---------------------------------------------------------------------------
// The same attention for MANY query tiles per stream (long sequences, many streams): one
// query tile per WAVE.  The 4 waves of a workgroup walk the key tiles together and share
// every K and V tile through LDS (fragment order is kept, a tile is copied 16 bytes per
// thread as it lies), so a stream's cache is read once per 128 queries instead of once per
// 32, and there is nothing to merge.  A wave skips the key tiles behind its last query.
// The statistic is parked for stats_reduce_kernel (this kernel is only used where that
// reduction applies): waves that hold text rows run the second pass over the vision keys,
// whose K tiles the workgroup stages the same way.
// ---------------------------------------------------------------------------
// (3 waves per SIMD: measured 11 % faster than the 236 registers the compiler takes if allowed)
template <int HD, bool F16>
__global__ __launch_bounds__(256, 3) void attn_rows4_kernel(AttnArgs a) {
  constexpr int NC = HD / 16;      // k-tiles of a head
  constexpr int NI = HD / 32;      // feature blocks of a head
  constexpr int TILE = NC * 64;    // 16-byte chunks of a K tile (and of a V tile)
  constexpr int PER = TILE / 256;  // chunks per thread
  constexpr int AHEAD = 2;         // key tiles on their way to LDS while one is worked on (1 and 3: no faster)
  constexpr int NBUF = AHEAD + 1;
  __shared__ uint4 kvs[NBUF][2][TILE];  // [buffer][K, V]
  __shared__ int s_text[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j = lane & 31, g = lane >> 5;
  // grid (heads, streams, query blocks): the query block is the slowest index, see below
  const int b = blockIdx.y, h = blockIdx.x;
  read_args(a.rows, a.qbuf, a.out, a.kc_out, a.kv, a.kv_stream_stride, a.n_q_heads, a.n_kv_heads, a.max_seq, a.L_v, a.L_t,
            a.scale_log2e, a.attn_mean, a.statp, a.TT, a.lv_pad, a.rows4_from);
  const int off_b = ld_scalar(a.slot_off + b);
  const int n_b = ld_scalar(a.slot_off + b + 1) - off_b;
  // the stream's query tiles are dealt to its workgroups in equal shares of at most 4 (33
  // tiles: 9 workgroups of 3 or 4, not 8 of 4 and one with a single busy wave)
  const int n_qt = (n_b + 31) >> 5, n_wg = (n_qt + 3) >> 2;
  if ((int)blockIdx.z >= n_wg || n_b < a.rows4_from) return;
  // The workgroups of the streams' LAST queries have the longest walks, and the launch lasts
  // as long as the last of them: they start first, those of ALL streams and heads before any
  // shorter one (the heads are the fastest index: workgroup id % 8, the XCD, is then the
  // same for all workgroups of a stream and head, which share its K and V in that L2).
  const int xb = n_wg - 1 - (int)blockIdx.z;
  const int qt_end = (xb + 1) * n_qt / n_wg;
  const int qt = xb * n_qt / n_wg + w, s0 = qt * 32;  // this wave's query tile
  const bool active = qt < qt_end;
  const int hk = h / (a.n_q_heads / a.n_kv_heads);
  const bool valid = active && s0 + j < n_b;
  const int sg = off_b + (valid ? s0 + j : n_b - 1);  // this lane's query slot
  const int pos = valid ? (a.rows[sg] & 0xffff) : 0;
  const int pos_last = active ? (a.rows[off_b + min(s0 + 31, n_b - 1)] & 0xffff) : -1;
  const int n_kt = (pos_last >> 5) + 1;  // 0 for a wave without queries
  const int pos_first = __builtin_amdgcn_readfirstlane(pos);  // lane 0: the wave's first query
  // rows ascend by position: the workgroup needs the key tiles of its last query
  const int pos_wg = ld_scalar(a.rows + off_b + min(qt_end * 32 - 1, n_b - 1)) & 0xffff;
  const int n_kt_wg = (pos_wg >> 5) + 1;

  const size_t head_elems = (size_t)a.max_seq * HD;
  const uint4* ksrc = (const uint4*)(a.kv + (size_t)b * a.kv_stream_stride + (size_t)hk * head_elems) + tid;
  const uint4* vsrc = ksrc + (size_t)a.n_kv_heads * head_elems / 8;

  uint4 qf[NC];
  {
    const bf16_t* qsrc = a.qbuf + ((size_t)(sg >> 5) * a.n_q_heads + h) * (size_t)NC * 512 +
                         (size_t)(((sg & 31) + 32 * g) << 3);
#pragma unroll
    for (int c = 0; c < NC; ++c) qf[c] = *(const uint4*)(qsrc + (size_t)c * 512);
  }
  f32x16 o[NI];
#pragma unroll
  for (int ib = 0; ib < NI; ++ib)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[ib][i] = 0.f;
  float m = -INFINITY, l = 0.f;

  // K and V tiles go global -> LDS directly (global_load_lds_dwordx4: lane l's 16 bytes
  // land at base + 16 l, so a wave copies 1 KiB as it lies), AHEAD tiles before they are
  // used, into a ring of AHEAD + 1 buffers: no staging registers, and the load latency is
  // spread over AHEAD tiles of work.  The copies are inline assembly, so the compiler does
  // not count them and the waits are placed by hand: loads return in issue order, every
  // tile is 2 PER copies per wave, nothing else is loaded inside the loop, and what was
  // loaded before it is older; so with the copies of AHEAD tiles issued, "at most
  // 2 PER (AHEAD - 1) outstanding" means that the oldest tile has landed.
  static_assert(PER == 1 || PER == 2, "a tile is 2 or 4 copies per wave");
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&kvs[0][0][w * 64]);
  auto copy_tile = [&](int kt, int buf) {
    const uint4* ks = ksrc + (size_t)kt * TILE;
    const uint4* vs = vsrc + (size_t)kt * TILE;
    const uint32_t d = lds0 + buf * (2 * TILE * 16);
    if (PER == 2) {
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %4, off\n\t"
          "s_mov_b32 m0, %1\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %5, off\n\t"
          "s_mov_b32 m0, %2\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %6, off\n\t"
          "s_mov_b32 m0, %3\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %7, off"
          :
          : "s"(d), "s"(d + 4096), "s"(d + TILE * 16), "s"(d + TILE * 16 + 4096), "v"(ks), "v"(ks + 256),
            "v"(vs), "v"(vs + 256)
          : "memory", "m0");
    } else {
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %2, off\n\t"
          "s_mov_b32 m0, %1\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %3, off"
          :
          : "s"(d), "s"(d + TILE * 16), "v"(ks), "v"(vs)
          : "memory", "m0");
    }
  };
  // (the query fragments are waited for here, so that no wait for them ends up inside the loop,
  // where it would wait for the copies as well)
#pragma unroll
  for (int c = 0; c < NC; ++c) asm volatile("" ::"v"(qf[c].x), "v"(qf[c].y), "v"(qf[c].z), "v"(qf[c].w));
#pragma unroll
  for (int t = 0; t < AHEAD; ++t) copy_tile(min(t, n_kt_wg - 1), t);
  for (int kt = 0; kt < n_kt_wg; ++kt) {
    const int buf = kt % NBUF;
    // tile kt has landed (this wave's part; the barrier makes that all four parts), and every
    // wave has left tile kt - 1, whose buffer takes tile kt + AHEAD
    constexpr int YOUNGER = 2 * PER * (AHEAD - 1);
    static_assert(YOUNGER == 0 || YOUNGER == 2 || YOUNGER == 4 || YOUNGER == 8, "add the wait for this count");
    if (YOUNGER == 8) VLAC_VMCNT(8);
    else if (YOUNGER == 4) VLAC_VMCNT(4);
    else if (YOUNGER == 2) VLAC_VMCNT(2);
    else VLAC_VMCNT(0);
    __syncthreads();
    copy_tile(min(kt + AHEAD, n_kt_wg - 1), (kt + AHEAD) % NBUF);
    if (kt < n_kt) {
      f32x16 s;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) s = mfma32<F16>(kvs[buf][0][c * 64 + lane], qf[c], s);
      // register 4*q4 + e of a lane is key 32*kt + 8*q4 + 4*g + e; only the tiles that
      // reach past the wave's first query need the causal mask
      float tmax = -INFINITY;
      if (32 * kt + 31 <= pos_first) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          s[i] *= a.scale_log2e;
          tmax = fmaxf(tmax, s[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int kp = 32 * kt + 8 * (i >> 2) + 4 * g + (i & 3);
          s[i] = (kp <= pos) ? s[i] * a.scale_log2e : -INFINITY;
          tmax = fmaxf(tmax, s[i]);
        }
      }
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
      // The reference point m of a query's exponentials follows its running maximum only
      // when that has grown by more than 8 (a factor of 256 in p, which fp16 operands and
      // fp32 sums hold easily): after the first tiles that is rare, and a tile in which no
      // query of the wave moves its reference skips the rescaling of the 64 accumulators.
      // (The decision is per query, so a query's result does not depend on its neighbours.)
      float alpha = 1.f;
      if (tmax > m + 8.f) {
        alpha = __builtin_amdgcn_exp2f(m - tmax);  // first tile: 2^-inf = 0
        m = tmax;
      }
      const float m_use = (m == -INFINITY) ? 0.f : m;
      float psum = 0.f;
      float pr[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        pr[i] = __builtin_amdgcn_exp2f(s[i] - m_use);
        psum += pr[i];
      }
      l = l * alpha + psum;
      const bool rescale = __any(alpha != 1.f);
      uint4 pb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        pb[t].x = pack_p2<F16>(pr[8 * t + 0], pr[8 * t + 1]);
        pb[t].y = pack_p2<F16>(pr[8 * t + 2], pr[8 * t + 3]);
        pb[t].z = pack_p2<F16>(pr[8 * t + 4], pr[8 * t + 5]);
        pb[t].w = pack_p2<F16>(pr[8 * t + 6], pr[8 * t + 7]);
      }
      if (rescale) {
#pragma unroll
        for (int ib = 0; ib < NI; ++ib)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[ib][i] *= alpha;
      }
#pragma unroll
      for (int ib = 0; ib < NI; ++ib) {
#pragma unroll
        for (int t = 0; t < 2; ++t) o[ib] = mfma32<F16>(kvs[buf][1][(ib * 2 + t) * 64 + lane], pb[t], o[ib]);
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy outlives the loop
  __syncthreads();                                  // (the buffers are used again below)
  l += __shfl_xor(l, 32);
  const float inv = 1.f / l;  // (a wave without queries: never used)
  if (valid) {
#pragma unroll
    for (int ib = 0; ib < NI; ++ib)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int f = h * HD + 32 * ib + 8 * q4 + 4 * g;
        *(uint2*)(a.out + frag_off(sg, f, a.kc_out)) =
            make_uint2(pack_op2<F16>(o[ib][4 * q4] * inv, o[ib][4 * q4 + 1] * inv),
                       pack_op2<F16>(o[ib][4 * q4 + 2] * inv, o[ib][4 * q4 + 3] * inv));
      }
  }

  // ---- text-to-vision statistic (the conditions up to the loop are uniform over the workgroup) ----
  if (!a.attn_mean || a.L_t <= 0 || a.L_v <= 0) return;
  if (pos_wg < a.L_v) return;  // no text row in this workgroup
  const int x_first = (n_b - a.L_t) >> 5;  // first query tile that holds a text row
  const bool text_wave = active && pos_last >= a.L_v;
  const bool is_text = valid && pos >= a.L_v;
  const int n_vt = (a.L_v + 31) >> 5;
  // The waves that hold text rows publish their query fragments, reference points and 1/sums
  // in LDS (all waves are past their last read of the buffers: the loop ended on a barrier);
  // then the 4 waves deal the vision key tiles of every such query tile among themselves,
  // each reading its K tiles straight from global memory: the workgroup with a stream's last
  // queries, which has the longest walk anyway, adds n_vt / 4 steps to it, not n_vt.
  uint4* q_sh = &kvs[0][0][0];                   // [4][NC][64]
  float* f_sh = (float*)(q_sh + 4 * NC * 64);    // [4][3][64]: reference point, 1/sum, text row?
  static_assert(4 * NC * 64 + 3 * 64 <= NBUF * 2 * TILE, "the buffers hold what the waves publish");
  if (text_wave) {
#pragma unroll
    for (int c = 0; c < NC; ++c) q_sh[(w * NC + c) * 64 + lane] = qf[c];
    f_sh[(w * 3 + 0) * 64 + lane] = m;
    f_sh[(w * 3 + 1) * 64 + lane] = is_text ? inv : 0.f;  // (a row that is no text row adds nothing)
    f_sh[(w * 3 + 2) * 64 + lane] = is_text ? 1.f : 0.f;
  }
  if (lane == 0) s_text[w] = text_wave ? 1 : 0;
  __syncthreads();
  const bf16_t* kbase = a.kv + (size_t)b * a.kv_stream_stride + (size_t)hk * head_elems + (size_t)lane * 8;
  auto load_k = [&](int kt, uint4(&kf)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *(const uint4*)(kbase + ((size_t)kt * NC + c) * 512);
  };
  // Here the scores are taken the other way round, Q K^T: a lane's column is a KEY and its 16
  // registers are queries (8 q4 + 4 g + e), so the sum over the queries of a tile is 16
  // additions in the lane and one exchange between the two halves of the wave.
  for (int tw = 0; tw < 4; ++tw) {
    if (!s_text[tw]) continue;
    uint4 qt_f[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) qt_f[c] = q_sh[(tw * NC + c) * 64 + lane];
    // per register: its query's reference point and 1/sum (0: no text row), read from LDS
    // where they are needed (they would cost 32 registers next to three K tiles)
    const float* m_q = f_sh + (tw * 3 + 0) * 64 + 4 * g;
    const float* inv_q = f_sh + (tw * 3 + 1) * 64 + 4 * g;
    float* park = a.statp + (((size_t)b * a.n_q_heads + h) * a.TT + (qt - w + tw - x_first)) * a.lv_pad;
    uint4 kf[NC], kn[NC];
    if (w < n_vt) load_k(w, kf);
    for (int kt = w; kt < n_vt; kt += 4) {
      if (kt + 4 < n_vt) load_k(kt + 4, kn);
      f32x16 s;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) s = mfma32<F16>(qt_f[c], kf[c], s);
      float r = 0.f;  // fixed order: the lane's 16 queries, then the other half's
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int qi = 8 * (i >> 2) + (i & 3);
        const float iq = inv_q[qi];
        r += iq != 0.f ? exp2f(s[i] * a.scale_log2e - m_q[qi]) * iq : 0.f;
      }
      r += __shfl_xor(r, 32);
      if (g == 0) park[32 * kt + j] = r;
#pragma unroll
      for (int c = 0; c < NC; ++c) kf[c] = kn[c];
    }
  }
}

// The statistic of all layers at once, after the last layer (text-to-vision attention
// averaged over heads and text queries, Eq. avistext): adds the sums that the attention
// kernels of the prefill parked, [layer][B][Hq][TT][lv_pad], over heads and text tiles in
// fixed order.  grid (layers, B, tokens / 64): the 4 waves of a workgroup take a quarter of the
// parked sums of 64 tokens each, 16 at a time, and meet in LDS (a thread that walked them all, 256
// tokens per workgroup and one workgroup per layer and stream: 24 us at 4 layers x 512 tokens, now
// 5.8; 8 streams x 1024 tokens 26 -> 5.4).
// slot_off is [layers][slot_stride] (first slot of every stream at every layer), from which the
// number of text tiles follows as in the kernel.
__global__ __launch_bounds__(256) void stats_reduce_kernel(const float* __restrict__ statp,
                                                           const int* __restrict__ slot_off,
                                                           int slot_stride, int B, int n_q_heads,
                                                           int TT, int lv_pad, int L_v, int L_t,
                                                           float* __restrict__ attn_mean) {
  __shared__ float sums[4][64];
  const int layer = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  read_args(statp, slot_off, slot_stride, B, n_q_heads, TT, lv_pad, L_v, L_t, attn_mean);
  const int* so = slot_off + (size_t)layer * slot_stride;
  const int n_b = ld_scalar(so + b + 1) - ld_scalar(so + b);
  const int x_first = (n_b - L_t) >> 5;
  const int n_tt = ((n_b - 1) >> 5) - x_first + 1;
  const int n_part = n_q_heads * n_tt, per = (n_part + 3) >> 2, p_end = min(n_part, (w + 1) * per);
  const float* part0 = statp + ((size_t)layer * B + b) * n_q_heads * TT * lv_pad;
  const float norm = 1.f / ((float)n_q_heads * (float)L_t);
  const int v = blockIdx.z * 64 + lane, vv = min(v, L_v - 1);
  float acc = 0.f;
  for (int p0 = w * per; p0 < p_end; p0 += 16) {
    float t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int p = min(p0 + i, p_end - 1), hh = p / n_tt, tq = p - hh * n_tt;
      t[i] = part0[((size_t)hh * TT + tq) * lv_pad + vv];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) acc += (p0 + i < p_end) ? t[i] : 0.f;
  }
  sums[w][lane] = acc;
  __syncthreads();
  if (w == 0 && v < L_v)
    attn_mean[((size_t)layer * B + b) * L_v + v] = (sums[0][lane] + sums[1][lane] + sums[2][lane] + sums[3][lane]) * norm;
}

static const size_t kDecLds = 144 * 1024;  // most that the waves of attn_decode_kernel exchange

int attn_init() {
  hipError_t e;
#define VLAC_SET(HD_, F16_)                                                                             \
  if ((e = hipFuncSetAttribute((const void*)attn_decode_kernel<HD_, F16_, false>,                        \
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDecLds)) != hipSuccess) return (int)e; \
  if ((e = hipFuncSetAttribute((const void*)attn_decode_kernel<HD_, F16_, true>,                         \
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDecLds)) != hipSuccess) return (int)e;
  VLAC_SET(128, true) VLAC_SET(128, false) VLAC_SET(64, true) VLAC_SET(64, false)
#undef VLAC_SET
  return 0;
}

bool attention_defers_stats(const vlac_ctx* c, int B, int L_v, int L_t) {
  // text rows of a stream lie in at most ceil(L_t / 32) + 1 tiles of 32 slots
  const int n_tt_max = (L_t + 31) / 32 + 1;
  const size_t need = (size_t)c->cfg.n_layers * B * c->cfg.n_q_heads * kStatDeferTT * round_up(L_v > 0 ? L_v : 1, 32);
  return L_t > 0 && L_v > 0 && n_tt_max <= kStatDeferTT && need <= c->statp_floats;
}

void launch_stats_reduce(vlac_ctx* c, int B, int L_v, int L_t, float* out_attn_mean, hipStream_t st) {
  hipLaunchKernelGGL(stats_reduce_kernel, dim3(c->cfg.n_layers, B, (L_v + 63) / 64), dim3(256), 0, st, c->statp,
                     c->slot_off, c->cfg.max_batch + 1, B, c->cfg.n_q_heads, kStatDeferTT,
                     round_up(L_v, 32), L_v, L_t, out_attn_mean);
}

void launch_attention(vlac_ctx* c, int layer, int B, int rows_cap_per_stream, int L_v, int L_t,
                      const int* rows, const int* slot_off, int decode_pos, bf16_t* kv,
                      float* out_attn_mean, hipStream_t st) {
  const vlac_model_cfg& m = c->cfg;
  AttnArgs a;
  a.rows = rows;
  a.slot_off = slot_off;
  a.decode_pos = decode_pos;
  a.qbuf = c->qbuf;
  a.out = c->xa;
  a.kc_out = c->kpad_q / 16;
  const size_t layer_elems = (size_t)2 * m.n_kv_heads * m.max_seq * m.head_dim;
  a.kv = kv + (size_t)layer * layer_elems;
  a.kv_stream_stride = (size_t)m.n_layers * layer_elems;
  a.n_q_heads = m.n_q_heads;
  a.n_kv_heads = m.n_kv_heads;
  a.max_seq = m.max_seq;
  a.L_v = L_v;
  a.L_t = L_t;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)m.head_dim);
  a.attn_mean = out_attn_mean ? out_attn_mean + (size_t)layer * B * L_v : nullptr;
  a.attn_mean_stride = L_v;
  a.lv_pad = round_up(L_v > 0 ? L_v : 1, 32);
  a.defer_stats = out_attn_mean && attention_defers_stats(c, B, L_v, L_t);
  if (a.defer_stats) {
    a.TT = kStatDeferTT;
    a.statp = c->statp + (size_t)layer * B * m.n_q_heads * kStatDeferTT * a.lv_pad;
  } else {
    a.TT = c->stat_tt;
    a.statp = c->statp;
  }
  a.stat_counters = c->stat_counters;
  if (decode_pos >= 0) {
    const int group = m.n_q_heads / m.n_kv_heads, nc = group < 32 ? group : 32;
    const int n_kt = (decode_pos >> 5) + 1;
    const size_t row = (size_t)nc * (m.head_dim + 4) * sizeof(float);  // LDS that a wave's part takes
    const bool multi = n_kt > kDecWaves || n_kt * row > kDecLds;
    int nw = multi ? kDecWavesMulti : n_kt;
    while (nw * row > kDecLds) --nw;
    const dim3 gridd(m.n_kv_heads * ((group + 31) / 32), B), block(64 * nw);
#define VLAC_DEC(HD_, F16_)                                                                                  \
  {                                                                                                         \
    if (multi) hipLaunchKernelGGL((attn_decode_kernel<HD_, F16_, true>), gridd, block, nw * row, st, a);    \
    else hipLaunchKernelGGL((attn_decode_kernel<HD_, F16_, false>), gridd, block, nw * row, st, a);         \
  }
    if (m.head_dim == 128) {
      if (c->f16) VLAC_DEC(128, true) else VLAC_DEC(128, false)
    } else {
      if (c->f16) VLAC_DEC(64, true) else VLAC_DEC(64, false)
    }
#undef VLAC_DEC
    return;
  }
  // Sequences of 256 tokens or more of many streams (work for every CU several times over;
  // 32 streams x 304 tokens of the grouped-query model: 29.4 against 30.5 ms per full
  // prefill): streams with more
  // than two query tiles to recompute (65 rows) go to the kernel with one query tile per
  // WAVE, where the 4 waves of a workgroup share K and V (the cache is read once per 128
  // queries and not once per 32: measured at 8 streams x 1056 tokens, 134 rows per stream:
  // 4.2 ms per 32-layer prefill outside the GEMMs against 5.7 ms); streams with fewer rows
  // (and every other shape) to the kernel with one query tile per workgroup and the key
  // tiles dealt to its waves, which has the shorter critical path.  The row counts are
  // known on the device only, so both kernels are launched and each leaves the other's
  // streams alone.
  const int groups = (rows_cap_per_stream + 127) / 128;
  a.rows4_from = 0;
  if (rows_cap_per_stream >= 256 && (long long)groups * m.n_q_heads * B >= 512 &&
      (!a.attn_mean || a.defer_stats)) {
    a.rows4_from = 65;
    dim3 grid4(m.n_q_heads, B, groups);
    if (m.head_dim == 128) {
      if (c->f16) hipLaunchKernelGGL((attn_rows4_kernel<128, true>), grid4, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((attn_rows4_kernel<128, false>), grid4, dim3(256), 0, st, a);
    } else {
      if (c->f16) hipLaunchKernelGGL((attn_rows4_kernel<64, true>), grid4, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((attn_rows4_kernel<64, false>), grid4, dim3(256), 0, st, a);
    }
  }
  // (beside the other kernel only streams of up to rows4_from - 1 rows are left to this one: two query tiles;
  // with a workgroup for every tile of every stream the idle launch takes 6.6 us at 8 x 1057 tokens, so 5.0)
  const int rows_most = a.rows4_from > 0 ? a.rows4_from - 1 : rows_cap_per_stream;
  dim3 grid(m.n_q_heads, (rows_most + 31) / 32, B);
  if (m.head_dim == 128) {
    if (c->f16) hipLaunchKernelGGL((attn_rows_kernel<128, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attn_rows_kernel<128, false>), grid, dim3(256), 0, st, a);
  } else {
    if (c->f16) hipLaunchKernelGGL((attn_rows_kernel<64, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attn_rows_kernel<64, false>), grid, dim3(256), 0, st, a);
  }
}
