// Front end for the visual tokens: the patch -> embedding projection, for the patches
// that the sparse prefill will recompute only (an extension of the token reuse of
// VLA-Cache, Sec. 3.2 / Alg. 2, to the step before the decoder: a token whose K/V are
// reused at the first layer needs no embedding either).  The projection is a fixed linear
// map of the patch's pixels, the stand-in used here for the vision encoder:
//   e[i, :] = (pixels_i / 127.5 - 1) . W,   pixels_i = patch i as [p rows][p cols][3] bytes.
//
// Work: (changed patches) x 3 p^2 x d multiply-adds against a matrix of a few MB that stays
// in L2, on the matrix cores: pixels / 127.5 - 1 = (2 pixels - 255) / 255, and 2 pixels - 255
// is an odd integer of at most 8 bits, which bf16 holds exactly, also divided by 256; so with
// bf16 weights every product (2 pixels - 255) / 256 x w is exact and only the fp32 sum rounds, as
// it did with fp32 multiply-adds, and nothing is larger on the way than at the end: finite
// results stay finite.  The patches to do are compacted into a list first, so that the work is
// proportional to their number.
#include <type_traits>

#include "common.h"

// list[b][0 .. n_live[b]) = the patches of stream b that are NOT among the first m reuse
// entries, ascending.  One workgroup per stream.  For calls of many workgroups, which would each spend 2 us on it
// (emb_own).
__global__ __launch_bounds__(256) void embed_mark_kernel(const int32_t* __restrict__ reuse_order,
                                                         const int32_t* __restrict__ reuse_count,
                                                         int stride, const int32_t* __restrict__ layer_count,
                                                         int n_layers, int L_v, uint8_t* __restrict__ flags,
                                                         int* __restrict__ list, int* __restrict__ n_live) {
  __shared__ int wsum[4];
  __shared__ int base;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint8_t* f = flags + (size_t)b * 4096;
  int* out = list + (size_t)b * 4096;
  for (int i = tid; i < L_v; i += 256) f[i] = 0;
  __syncthreads();
  if (reuse_order) {
    int m = min(max(reuse_count[b], 0), stride);
    if (layer_count) m = min(m, max(layer_count[(size_t)b * n_layers], 0));
    for (int i = tid; i < m; i += 256) {
      const int t = reuse_order[(size_t)b * stride + i];
      if (t >= 0 && t < L_v) f[t] = 1;
    }
  }
  if (tid == 0) base = 0;
  __syncthreads();
  for (int i0 = 0; i0 < L_v; i0 += 256) {  // ordered compaction, 256 patches at a time
    const int i = i0 + tid;
    const bool live = i < L_v && !f[i];
    const unsigned long long mask = __ballot(live);
    if (lane == 0) wsum[w] = __popcll(mask);
    __syncthreads();
    int off = base;
    for (int k = 0; k < w; ++k) off += wsum[k];
    if (live) out[off + __popcll(mask & ((1ull << lane) - 1))] = i;
    __syncthreads();
    if (tid == 0) base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  if (tid == 0) n_live[b] = base;
}

struct EmbedReuse { const int32_t *order, *count; int stride; const int32_t* layer_count; int n_layers; };

// The patches [g0, g0 + PB) of that list, worked out by the workgroup itself; returns the list's length.  flags:
// L_v bytes of LDS that are used for nothing else until then.  (One round of workgroups: one launch less, 2.3 us of the
// GPU and 4 of the host; a front end of 256 patches, whose launches the host queues no faster than the GPU runs them,
// 40.0 -> 37.2 us.)
template <int PB>
__device__ __forceinline__ int embed_group(const EmbedReuse& r, int b, int L_v, int g0, uint8_t* flags, int* group) {
  __shared__ int wsum[2][4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i = tid * 4; i < L_v; i += 1024) *(uint32_t*)(flags + i) = 0;  // (the buffer is longer than L_v)
  __syncthreads();
  if (r.order) {
    int m = min(max(ld_scalar(r.count + b), 0), r.stride);
    if (r.layer_count) m = min(m, max(ld_scalar(r.layer_count + (size_t)b * r.n_layers), 0));
    for (int i = tid; i < m; i += 256) {
      const int t = r.order[(size_t)b * r.stride + i];
      if (t >= 0 && t < L_v) flags[t] = 1;
    }
  }
  __syncthreads();
  int base = 0;
  for (int i0 = 0, turn = 0; i0 < L_v; i0 += 256, turn ^= 1) {
    const int i = i0 + tid;
    const bool live = i < L_v && !flags[i];
    const unsigned long long mask = __ballot(live);
    if (lane == 0) wsum[turn][w] = __popcll(mask);
    __syncthreads();
    int at = base - g0 + __popcll(mask & ((1ull << lane) - 1));
    for (int k = 0; k < w; ++k) at += wsum[turn][k];
    if (live && at >= 0 && at < PB) group[at] = i;
    base += wsum[turn][0] + wsum[turn][1] + wsum[turn][2] + wsum[turn][3];
  }
  __syncthreads();
  return base;
}

typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(1)));

// Workgroup (x: 512 / KS output features, y: group of 32 RT live patches, z: stream).  The pixels
// of the group go to LDS as bf16 operands in fragment order ([k/16][lane] of 16 bytes, lane =
// patch + 32 (k/8 % 2)).  KS = 1: a wave multiplies them by 128 features of its own; KS = 4: the
// waves share 128 features, take a quarter of the k-tiles each, and their sums meet in LDS, which
// gives a small call four times the workgroups and a quarter of the chain.
// TWO: few patches of an even width in a frame at an even address, see the staging.
// A wave's operand tile t (of 4) covers the features 4 j + t, j = lane % 32: a lane then reads
// 4 neighbouring features of a weight row with one 8-byte load (w_proj is [k][feature], so the 8
// values of k that an operand wants are 8 loads, 8 rows of it, and two byte permutations per
// pair), and writes 4 neighbouring features of an embedding row with one 16-byte store.
// Bound by latency at one stream and by staging the pixels and writing the output at many.
// Measured at d_model 4096, 14 x 14 patches, kernel alone, against the fp32 multiply-adds of 8
// patches per workgroup that this replaces: 166 patches of one stream 12 us (42 before),
// 4800 patches of 8 streams 66 us (537 before; 192 with KS = 4 and two row tiles, which stages
// the same pixels 32 times).
// The pixels come by 16-byte loads at any address and the weights by a scalar address per k-tile: d_model 4096,
// 8 x 1024 patches 70 -> 67 us of 14 x 14 pixels, front end 115 -> 112; 16 x 16 179 -> 168; 16 x 1024 of 13 x 13
// (2-byte loads at even rows, single bytes at the odd ones before) 198 -> 165.  The phases of a workgroup add up:
// staging 13 us, products 28, output 15 of the 67 at 8 x 1024.
// (EMB_D k-tiles of weights in flight per wave: with 2 row tiles only 2, so that a
// second workgroup fits the CU: 85 -> 72 us per call at 8 x 1024 patches)
// OWN: the workgroup works the list out for itself, list and n_live are not read.
template <int RT, int KS, bool VEC, bool TWO, bool OWN>
__device__ __forceinline__ void embed_patches(const uint8_t* __restrict__ frame, int H, int W, int patch,
                                              const bf16_t* __restrict__ w_proj, int d, const int* __restrict__ list,
                                              const int* __restrict__ n_live, const EmbedReuse& reuse,
                                              float* __restrict__ embeds, int L) {
  extern __shared__ uint4 px[];  // [RT][k-tiles][64]; KS = 4: then, per row tile, the waves' sums
  constexpr int PB = 32 * RT, EMB_D = RT == 2 ? 2 : 4;
  const int gw = W / patch, dp = 3 * patch * patch, prow = 3 * patch, n_kt = (dp + 15) >> 4;
  const int b = blockIdx.z, g0 = blockIdx.y * PB, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int nl;
  const int* mine;
  if constexpr (OWN) {
    __shared__ int group[PB];
    nl = embed_group<PB>(reuse, b, gw * (H / patch), g0, (uint8_t*)px, group);
    mine = group;
  } else {
    nl = n_live[b];
    mine = list + (size_t)b * 4096 + g0;
  }
  if (g0 >= nl) return;
  const int cnt = min(PB, nl - g0);
  const int j = lane & 31, g = lane >> 5;
  const int f0 = (KS == 1 ? blockIdx.x * 512 + 128 * w : blockIdx.x * 128) + 4 * j;  // this lane's 4 features
  const int fl = min(f0, d - 4);                                                     // (d is a multiple of 32)

  // this wave's k-tiles [kt0, kt1); past the last weight row it is read again (see the pixels)
  const int kt0 = KS == 1 ? 0 : w * n_kt / 4, kt1 = KS == 1 ? n_kt : (w + 1) * n_kt / 4;
  uint2 wb[EMB_D][8];
  // (a scalar address per k-tile and the lane's offsets of its 8 rows, the last k-tile's beside the
  // others': the loop multiplies nothing)
  uint32_t off[8], off_last[8];
  const uint32_t off_max = 2u * ((uint32_t)(dp - 1 - (n_kt - 1) * 16) * (uint32_t)d + (uint32_t)fl);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    off[u] = u == 0 ? 2u * ((uint32_t)(8 * g) * (uint32_t)d + (uint32_t)fl) : off[u - 1] + 2u * (uint32_t)d;
    off_last[u] = min(off[u], off_max);
  }
  auto load_w = [&](int kt, uint2(&x)[8]) {
    const char* base = (const char*)(w_proj + (size_t)kt * 16 * d);
    const bool last = kt == n_kt - 1;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bf16_t* src = (const bf16_t*)(base + (last ? off_last[u] : off[u]));
      if constexpr (VEC) x[u] = *(const uint2*)src;
      else x[u] = make_uint2(src[0] | ((uint32_t)src[1] << 16), src[2] | ((uint32_t)src[3] << 16));
    }
  };
  auto first_weights = [&]() {
#pragma unroll
    for (int s = 0; s < EMB_D; ++s) load_w(min(kt0 + s, n_kt - 1), wb[s]);
  };

  // pixels: every thread has one patch of the group; unused patches of the group stay undefined (an
  // operand row only reaches its own result row)
  uint16_t* px16 = (uint16_t*)px;
  auto odd = [](uint32_t v) { return fmaf(1.f / 128.f, (float)v, -255.f / 256.f); };  // (2 v - 255) / 256, exact
  {
    constexpr int STEP = 256 / PB;
    const int p = tid % PB, q0 = tid / PB;
    const int i = mine[min(p, cnt - 1)], r = i / gw, c = i - r * gw;
    const size_t pitch = (size_t)W * 3;
    const uint8_t* src = frame + ((size_t)b * H + (size_t)r * patch) * pitch + (size_t)c * prow;
    uint16_t* dst = px16 + (size_t)(p >> 5) * n_kt * 512 + (p & 31) * 8;
    auto at = [&](int k) { return dst + ((k >> 3) << 8) + (k & 7); };
    // 16 bytes at a time, at whatever address (the last ones of a pixel row end with it and overlap those
    // before), several loads in flight; PAIRS: two pixels per store (even patches: every row starts at an
    // even k).  The first weights are asked for behind the first pixels, which are used first.
    auto stage = [&](auto pairs) {
      constexpr int U = RT == 1 ? 6 : 4;  // (loads in flight: 14 x 14 pixels in three groups, 13 x 13 of few patches at once)
      const int n_ch = (prow + 15) >> 4, n_q = patch * n_ch, inv = (65536 + n_ch - 1) / n_ch;  // (n_q <= 130)
      u32x4_u v[U];
      int k[U];
      auto load = [&](int q) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int t = min(q + u * STEP, n_q - 1), y = (t * inv) >> 16, x = min((t - y * n_ch) * 16, prow - 16);
          k[u] = y * prow + x;
          v[u] = *(const u32x4_u*)(src + y * pitch + x);
        }
      };
      auto store = [&](int q) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p < cnt && q + u * STEP < n_q) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              const uint32_t two = v[u][t >> 1] >> (16 * (t & 1));
              const uint32_t lo = __float_as_uint(odd(two & 255u)), hi = __float_as_uint(odd((two >> 8) & 255u));
              if constexpr (decltype(pairs)::value) {
                *(uint32_t*)at(k[u] + 2 * t) = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
              } else {
                *at(k[u] + 2 * t) = (uint16_t)(lo >> 16);
                *at(k[u] + 2 * t + 1) = (uint16_t)(hi >> 16);
              }
            }
          }
      };
      load(q0);
      __builtin_amdgcn_sched_barrier(0);
      first_weights();
      __builtin_amdgcn_sched_barrier(0);
      store(q0);
      for (int q = q0 + U * STEP; q < n_q; q += U * STEP) {
        load(q);
        store(q);
      }
    };
    if constexpr (TWO) {
      // (few patches of rows on even addresses: two-byte loads, seven in flight, behind the first weights, in an
      // instance of their own.  166 patches of one stream 10.0 -> 9.6 us, 12 streams of 90 patches 20.4 -> 19.7
      // against one instance with both ways in it, whose 224 registers are 172 here; with the 16-byte loads 10.9 and 23.2)
      first_weights();
      for (int y = q0; y < patch && p < cnt; y += STEP) {
        const uint8_t* row = src + y * pitch;
        const int k0 = y * prow;
        int x = 0;
        for (; x + 14 <= prow; x += 14) {
          uint16_t v[7];
#pragma unroll
          for (int u = 0; u < 7; ++u) v[u] = *(const uint16_t*)(row + x + 2 * u);
#pragma unroll
          for (int u = 0; u < 7; ++u)
            *(uint32_t*)at(k0 + x + 2 * u) = __builtin_amdgcn_perm(__float_as_uint(odd((uint32_t)v[u] >> 8)),
                                                                   __float_as_uint(odd((uint32_t)v[u] & 255u)), 0x07060302u);
        }
        for (; x < prow; ++x) *at(k0 + x) = (uint16_t)(__float_as_uint(odd(row[x])) >> 16);
      }
    } else if (prow >= 16) {
      if (patch & 1) stage(std::false_type{});
      else stage(std::true_type{});
    } else {
      first_weights();
      for (int y = q0; y < patch && p < cnt; y += STEP)
        for (int x = 0; x < prow; ++x) *at(y * prow + x) = (uint16_t)(__float_as_uint(odd(src[y * pitch + x])) >> 16);
    }
  }
  if (const int n_pad = n_kt * 16 - dp; n_pad > 0) {
    // k past the last pixel: the last weight row is read again there, and the last pixel's value x is
    // dealt over its own place and those (x / 2, x / 4, ..., the last two alike, all exact).  Zeros
    // would do for finite weights, but infinity times zero is not a number.  (Zeros for the weights
    // as well, chosen at the loads or ahead of the last k-tile: 85 and 68 us against 66 at 4800 patches.)
    __syncthreads();
    if (tid < cnt) {
      uint16_t* dst = px16 + (size_t)(tid >> 5) * n_kt * 512 + (tid & 31) * 8;
      uint16_t x = 0;
      for (int k = dp - 1; k < n_kt * 16; ++k) {
        uint16_t* at = dst + (k >> 4) * 512 + ((k >> 3) & 1) * 256 + (k & 7);
        if (k == dp - 1) x = *at;
        if (k + 1 < n_kt * 16) x -= 1 << 7;  // half of it
        *at = x;
      }
    }
  }
  __syncthreads();

  f32x16 acc[RT][4];
#pragma unroll
  for (int m = 0; m < RT; ++m)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[m][t][i] = 0.f;
  auto step = [&](int kt, uint2(&x)[8]) {
    // operand of tile t: the 8 values of k of feature 4 j + t, a half of a dword per weight row
    uint4 op[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t sel = (t & 1) ? 0x07060302u : 0x05040100u;
      uint32_t v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t lo = (t >> 1) ? x[2 * q].y : x[2 * q].x;
        const uint32_t hi = (t >> 1) ? x[2 * q + 1].y : x[2 * q + 1].x;
        v[q] = __builtin_amdgcn_perm(hi, lo, sel);
      }
      op[t] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_w(min(kt + EMB_D, n_kt - 1), x);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < RT; ++m) {
      const uint4 q = px[((size_t)m * n_kt + kt) * 64 + lane];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[m][t] = mfma32<false>(q, op[t], acc[m][t]);
    }
  };
  // (whole groups without a branch inside, so that the loads of EMB_D k-tiles stay in flight)
  int kt = kt0;
  for (; kt + EMB_D <= kt1; kt += EMB_D) {
#pragma unroll
    for (int s = 0; s < EMB_D; ++s) step(kt + s, wb[s]);
  }
#pragma unroll
  for (int s = 0; s < EMB_D - 1; ++s)
    if (kt + s < kt1) step(kt + s, wb[s]);

  auto store = [&](int p, float4 s) {
    if (p < cnt && f0 < d) {
      float* out = embeds + ((size_t)b * L + mine[p]) * d + f0;
      constexpr float one = 255.f / 256.f;
      s.x /= one; s.y /= one; s.z /= one; s.w /= one;
      if constexpr (VEC) {
        *(float4*)out = s;
      } else {
        out[0] = s.x; out[1] = s.y; out[2] = s.z; out[3] = s.w;
      }
    }
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int m = 0; m < RT; ++m)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        store(32 * m + 8 * (i >> 2) + 4 * g + (i & 3), make_float4(acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]));
    return;
  }
  // KS = 4: wave w finishes the registers 4 w .. 4 w + 3 of every tile (patches 8 w + 4 g + e), so
  // that all four waves store; the others' parts go through LDS, [wave][register][lane][tile]
  float* part = (float*)px;
#pragma unroll
  for (int m = 0; m < RT; ++m) {
    __syncthreads();  // (the pixels, or the sums of the row tile before, are no longer read)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if ((i >> 2) != w)
        *(float4*)(part + (((size_t)w * 16 + i) * 64 + lane) * 4) =
            make_float4(acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if ((i >> 2) != w) continue;
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {  // fixed order
        const float4 q = ww == w ? make_float4(acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i])
                                 : *(const float4*)(part + (((size_t)ww * 16 + i) * 64 + lane) * 4);
        s.x += q.x; s.y += q.y; s.z += q.z; s.w += q.w;
      }
      store(32 * m + 8 * (i >> 2) + 4 * g + (i & 3), s);
    }
  }
}

template <int RT, int KS, bool VEC, bool TWO>
__global__ __launch_bounds__(256, 2) void embed_patches_kernel(const uint8_t* __restrict__ frame, int H, int W, int patch,
                                                               const bf16_t* __restrict__ w_proj, int d,
                                                               const int* __restrict__ list, const int* __restrict__ n_live,
                                                               EmbedReuse reuse, float* __restrict__ embeds, int L) {
  embed_patches<RT, KS, VEC, TWO, KS == 4>(frame, H, W, patch, w_proj, d, list, n_live, reuse, embeds, L);
}

// the form of few patches with the list of embed_mark_kernel
template <bool VEC, bool TWO>
__global__ __launch_bounds__(256, 2) void embed_listed_kernel(const uint8_t* __restrict__ frame, int H, int W, int patch,
                                                              const bf16_t* __restrict__ w_proj, int d,
                                                              const int* __restrict__ list, const int* __restrict__ n_live,
                                                              float* __restrict__ embeds, int L) {
  embed_patches<1, 4, VEC, TWO, false>(frame, H, W, patch, w_proj, d, list, n_live, EmbedReuse{}, embeds, L);
}

// LDS: the pixel operands of the group; KS = 4: or the four waves' sums of one row tile
static size_t embed_lds(int RT, int KS, int dp) {
  return std::max((size_t)RT * ((dp + 15) / 16) * 1024, KS == 1 ? (size_t)0 : (size_t)65536);
}

int embed_init() {
  hipError_t e;
#define VLAC_EMB_SET(RT_, KS_, VEC_, TWO_)                                                               \
  if ((e = hipFuncSetAttribute((const void*)embed_patches_kernel<RT_, KS_, VEC_, TWO_>,                   \
                               hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024)) != hipSuccess) return (int)e;
  VLAC_EMB_SET(1, 4, true, true) VLAC_EMB_SET(1, 4, false, true) VLAC_EMB_SET(1, 4, true, false)
  VLAC_EMB_SET(1, 4, false, false) VLAC_EMB_SET(2, 1, true, false) VLAC_EMB_SET(2, 1, false, false)
#undef VLAC_EMB_SET
  for (const void* k : {(const void*)embed_listed_kernel<true, true>, (const void*)embed_listed_kernel<false, true>,
                        (const void*)embed_listed_kernel<true, false>, (const void*)embed_listed_kernel<false, false>})
    if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024)) != hipSuccess) return (int)e;
  return 0;
}

// Workgroups of 512 features and 64 patches from the size on at which they fill the chip once
// (256 of them; the number of live patches is known on the device only, so all are counted), and
// patches of up to 14 x 14 pixels, two groups of which fit the LDS of a CU (15 x 15: 86 KiB each).  Both sides, per call: at
// 128 such workgroups (4 x 256 patches, d_model 4096) 29 us against 22 with KS = 4, at 256 (2 x
// 1024) 33 against 38, at 1024 (8 x 1024) 85 against 117.
static const long long kEmbWide = 256;
// Workgroups of 128 features and 32 patches work the list of live patches out for themselves up to a round and a half of
// them where two fit a CU (patches of up to 20 x 20 pixels), up to two rounds where one does; more of them read it from
// embed_mark_kernel.  Front end, list by the launch and by the workgroups, us: 256 workgroups (1 x 256 patches, d_model
// 4096) 39.2 and 36.6; 512 (8 x 63) 43.0 and 41.0; 640 (1 x 625) 71.0 and 69.2; 768 (3 x 256) 43.2 and 41.7, (12 x 1024 of
// 16 x 16 pixels, d_model 256) 73.0 and 72.5; 1024 (4 x 256) 43.6 and 45.2; 1152 (12 x 90) 51.2 and 53.8; 1536 (6 x 256)
// 53.3 and 54.3; 8192 (8 x 1024 of 16 x 16) 172 and 193; 32768 (32 x 1024) 607 and 700.  26 x 26 pixels: 576 workgroups (1
// x 576) 86.4 and 85.1; 768 (12 x 1024, d_model 256) 133 and 136; 1024 (1 x 1024) 123 and 127.
static long long emb_own(size_t lds) { return lds <= 80 * 1024 ? 768 : 512; }

void launch_embed_patches(vlac_ctx* c, const uint8_t* frame, int B, int H, int W, int patch,
                          const bf16_t* w_proj, const int32_t* reuse_order, const int32_t* reuse_count,
                          int stride, const int32_t* layer_count, float* embeds, int L, hipStream_t st) {
  const int L_v = (H / patch) * (W / patch), d = c->cfg.d_model, dp = 3 * patch * patch;
  const EmbedReuse reuse = {reuse_order, reuse_count, stride, layer_count, c->cfg.n_layers};
  const bool wide = (long long)((d + 511) / 512) * ((L_v + 63) / 64) * B >= kEmbWide && embed_lds(2, 1, dp) <= 80 * 1024;
  const bool own = !wide && (long long)((d + 127) / 128) * ((L_v + 31) / 32) * B <= emb_own(embed_lds(1, 4, dp));
  // (8-byte weight loads and 16-byte stores where the caller's buffers allow them)
  const bool vec = (uintptr_t)w_proj % 8 == 0 && (uintptr_t)embeds % 16 == 0;
  const bool two = (patch & 1) == 0 && ((uintptr_t)frame & 1) == 0;
  if (!own)
    hipLaunchKernelGGL(embed_mark_kernel, dim3(B), dim3(256), 0, st, reuse_order, reuse_count, stride,
                       layer_count, c->cfg.n_layers, L_v, c->flags, c->embed_list, c->embed_n);
#define VLAC_EMB_GRID(RT_, KS_) \
  dim3((d + 512 / KS_ - 1) / (512 / KS_), (L_v + 32 * RT_ - 1) / (32 * RT_), B), dim3(256), embed_lds(RT_, KS_, dp), st
#define VLAC_EMB(RT_, KS_, VEC_, TWO_)                                                                                \
  hipLaunchKernelGGL((embed_patches_kernel<RT_, KS_, VEC_, TWO_>), VLAC_EMB_GRID(RT_, KS_), frame, H, W, patch, w_proj, \
                     d, c->embed_list, c->embed_n, reuse, embeds, L)
#define VLAC_EMB_FEW(VEC_, TWO_)                                                                                     \
  if (own) VLAC_EMB(1, 4, VEC_, TWO_);                                                                               \
  else hipLaunchKernelGGL((embed_listed_kernel<VEC_, TWO_>), VLAC_EMB_GRID(1, 4), frame, H, W, patch, w_proj, d,      \
                          c->embed_list, c->embed_n, embeds, L)
  if (wide) {
    if (vec) VLAC_EMB(2, 1, true, false); else VLAC_EMB(2, 1, false, false);
  } else if (two) {
    if (vec) { VLAC_EMB_FEW(true, true); } else { VLAC_EMB_FEW(false, true); }
  } else {
    if (vec) { VLAC_EMB_FEW(true, false); } else { VLAC_EMB_FEW(false, false); }
  }
#undef VLAC_EMB_FEW
#undef VLAC_EMB_GRID
#undef VLAC_EMB
}
